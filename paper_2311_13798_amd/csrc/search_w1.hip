// search_w1.hip -- the search kernels of width class 1 (sub-branches of at most 64 vertices).
#include "search_kernel.h"

namespace ebb {

template hipError_t search_launch<1>(bool, const SearchArgs&, int, int, hipStream_t);
template int64_t search_blocks<1>(bool, int64_t, int, int);
template hipError_t search_tables<1>(hipStream_t);

}  // namespace ebb
