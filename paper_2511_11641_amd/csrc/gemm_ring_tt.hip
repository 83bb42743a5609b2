// The contraction kernel for dY^T X (both operands K-slow: weight gradients), with and without the column sums of dY.
#include "gemm_ring.h"

#define TT_SHAPES(X) X(0, 256, 256, 2) X(1, 192, 256, 2) X(2, 256, 192, 2) X(3, 128, 256, 3) X(4, 256, 128, 3) X(5, 192, 192, 3) X(6, 128, 192, 3) X(7, 192, 128, 3) X(8, 128, 128, 4) X(9, 64, 128, 4)
#define TT_INST(I, BM, BN, NS)                                                                                   \
  template __global__ void gemm_bf16_ring_kernel<BM, BN, NS, true, true, false, GEMM_EPIS_TX>(const RingGrid, const GemmDesc); \
  template __global__ void gemm_bf16_ring_kernel<BM, BN, NS, true, true, true, GEMM_EPIS_TX>(const RingGrid, const GemmDesc);
TT_SHAPES(TT_INST)
template __global__ void gemm_bf16_ring_kernel<128, 128, 4, true, true, false, GEMM_EPIS_TX, true>(const RingGrid, const GemmDesc);
template __global__ void gemm_bf16_ring_kernel<128, 128, 4, true, true, true, GEMM_EPIS_TX, true>(const RingGrid, const GemmDesc);

hipError_t gemm_ring_launch_tt(ecospa_ctx* ctx, const GemmDesc& d, int shape, int k_chunk) {
#define TT_CASE(I, BM, BN, NS)                                                                                   \
  if (shape == I) return d.colsum ? ring_launch_shape<BM, BN, NS, true, true, true, GEMM_EPIS_TX>(ctx, d, k_chunk)   \
                                  : ring_launch_shape<BM, BN, NS, true, true, false, GEMM_EPIS_TX>(ctx, d, k_chunk);
  if (ring_wide(d) && shape == GEMM_RING_WIDE_SHAPE)
    return d.colsum ? ring_launch_shape<128, 128, 4, true, true, true, GEMM_EPIS_TX, true>(ctx, d, k_chunk)
                    : ring_launch_shape<128, 128, 4, true, true, false, GEMM_EPIS_TX, true>(ctx, d, k_chunk);
  TT_SHAPES(TT_CASE)
  return hipErrorInvalidValue;
}
