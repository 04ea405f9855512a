// FP64 instantiations of the Dslash kernels, three-hop links with all 18 reals.
#include "dslash_kernel.h"

namespace stag {

template hipError_t dslash_pc<P64, false>(const DslashArgs&, int, int, int, int, int, int, int, int, const DslashShape&, bool,
                                        size_t, hipStream_t);

}  // namespace stag
