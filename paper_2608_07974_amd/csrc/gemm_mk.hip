// The GEMM kernels of one operand layout (A MN-major, B K-major): a file each, so that they
// compile in parallel.
#include "gemm_tiles.h"

namespace zl {

template hipError_t run_layout<false, true>(const GemmDesc&, const EpiArgs&, hipStream_t, const char**);

}  // namespace zl
