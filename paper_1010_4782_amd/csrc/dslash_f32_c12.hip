// FP32 instantiations of the Dslash kernels, three-hop links with two rows.
#include "dslash_kernel.h"

namespace stag {

template hipError_t dslash_pc<P32, true>(const DslashArgs&, int, int, int, int, int, int, int, int, const DslashShape&, bool,
                                        size_t, hipStream_t);

}  // namespace stag
