// GEMM kernels of the input-gradient (dX = dY W^T) and LM-head layout (a file of its own: the layouts compile in parallel).
#include "gemm_kernel.h"

namespace bt {
void gemm_launch_nt(const GemmParams& p, int tile, bool wide, unsigned blocks, hipStream_t s) {
  launch_gemm<true, true>(p, tile, wide, blocks, s);
}
}  // namespace bt
