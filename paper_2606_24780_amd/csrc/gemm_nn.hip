// GEMM kernels of the forward (Y = X W) layout (a file of its own: the layouts compile in parallel).
#include "gemm_kernel.h"

namespace bt {
void gemm_launch_nn(const GemmParams& p, int tile, bool wide, unsigned blocks, hipStream_t s) {
  launch_gemm<true, false>(p, tile, wide, blocks, s);
}
}  // namespace bt
