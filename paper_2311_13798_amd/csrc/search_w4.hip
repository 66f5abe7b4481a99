// search_w4.hip -- the search kernels of width class 4 (sub-branches of at most 256 vertices).
#include "search_kernel.h"

namespace ebb {

template hipError_t search_launch<4>(bool, const SearchArgs&, int, int, hipStream_t);
template int64_t search_blocks<4>(bool, int64_t, int, int);
template hipError_t search_tables<4>(hipStream_t);

}  // namespace ebb
