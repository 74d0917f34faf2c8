// The GEMM kernels of one operand layout (A MN-major, B MN-major): a file each, so that they
// compile in parallel.
#include "gemm_tiles.h"

namespace zl {

template hipError_t run_layout<false, false>(const GemmDesc&, const EpiArgs&, hipStream_t, const char**);
template hipError_t run_pair_layout<false, false>(const GemmDesc&, const EpiArgs&, const GemmDesc&,
                                                  const EpiArgs&, hipStream_t, bool*);

}  // namespace zl
