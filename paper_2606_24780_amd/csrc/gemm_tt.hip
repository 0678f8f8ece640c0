// GEMM kernels of the doubly transposed layout (a file of its own: the layouts compile in parallel).
#include "gemm_kernel.h"

namespace bt {
void gemm_launch_tt(const GemmParams& p, int tile, bool wide, unsigned blocks, hipStream_t s) {
  launch_gemm<false, true>(p, tile, wide, blocks, s);
}
}  // namespace bt
