// search_w2.hip -- the search kernels of width class 2 (sub-branches of at most 128 vertices).
#include "search_kernel.h"

namespace ebb {

template hipError_t search_launch<2>(bool, const SearchArgs&, int, int, hipStream_t);
template int64_t search_blocks<2>(bool, int64_t, int, int);
template hipError_t search_tables<2>(hipStream_t);

}  // namespace ebb
