// search_w3.hip -- the search kernels of width class 3 (sub-branches of at most 192 vertices).
#include "search_kernel.h"

namespace ebb {

template hipError_t search_launch<3>(bool, const SearchArgs&, int, int, hipStream_t);
template int64_t search_blocks<3>(bool, int64_t, int, int);
template hipError_t search_tables<3>(hipStream_t);

}  // namespace ebb
