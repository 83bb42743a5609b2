// The contraction kernel for x W^T (both operands K-contiguous), 256- and 192-row tiles; every epilogue.
#include "gemm_ring.h"

#define NT_SHAPES(X) X(0, 256, 256, 2) X(1, 192, 256, 2) X(2, 256, 192, 2) X(4, 256, 128, 3)
#define NT_INST(I, BM, BN, NS) template __global__ void gemm_bf16_ring_kernel<BM, BN, NS, false, false, false, GEMM_EPIS_NT>(const RingGrid, const GemmDesc);
NT_SHAPES(NT_INST)

hipError_t gemm_ring_launch_nt_small(ecospa_ctx* ctx, const GemmDesc& d, int shape, int k_chunk);

hipError_t gemm_ring_launch_nt(ecospa_ctx* ctx, const GemmDesc& d, int shape, int k_chunk) {
#define NT_CASE(I, BM, BN, NS) if (shape == I) return ring_launch_shape<BM, BN, NS, false, false, false, GEMM_EPIS_NT>(ctx, d, k_chunk);
  NT_SHAPES(NT_CASE)
  return gemm_ring_launch_nt_small(ctx, d, shape, k_chunk);
}
