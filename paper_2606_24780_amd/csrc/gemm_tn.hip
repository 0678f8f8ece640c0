// GEMM kernels of the weight-gradient (dW = X^T dY) layout (a file of its own: the layouts compile in parallel).
#include "gemm_kernel.h"

namespace bt {
void gemm_launch_tn(const GemmParams& p, int tile, bool wide, unsigned blocks, hipStream_t s) {
  launch_gemm<false, false>(p, tile, wide, blocks, s);
}
}  // namespace bt
