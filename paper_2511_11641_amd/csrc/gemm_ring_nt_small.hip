// The contraction kernel for x W^T, the narrower tiles (a file of its own only to compile in parallel).
#include "gemm_ring.h"

#define NT_SHAPES(X) X(3, 128, 256, 3) X(5, 192, 192, 3) X(6, 128, 192, 3) X(7, 192, 128, 3) X(8, 128, 128, 4) X(9, 64, 128, 4) X(10, 128, 64, 4) X(11, 64, 64, 4)
#define NT_INST(I, BM, BN, NS) template __global__ void gemm_bf16_ring_kernel<BM, BN, NS, false, false, false, GEMM_EPIS_NT>(const RingGrid, const GemmDesc);
NT_SHAPES(NT_INST)
template __global__ void gemm_bf16_ring_kernel<128, 128, 4, false, false, false, GEMM_EPIS_NT, true>(const RingGrid, const GemmDesc);

hipError_t gemm_ring_launch_nt_small(ecospa_ctx* ctx, const GemmDesc& d, int shape, int k_chunk) {
#define NT_CASE(I, BM, BN, NS) if (shape == I) return ring_launch_shape<BM, BN, NS, false, false, false, GEMM_EPIS_NT>(ctx, d, k_chunk);
  if (ring_wide(d) && shape == GEMM_RING_WIDE_SHAPE) return ring_launch_shape<128, 128, 4, false, false, false, GEMM_EPIS_NT, true>(ctx, d, k_chunk);
  NT_SHAPES(NT_CASE)
  return hipErrorInvalidValue;
}
