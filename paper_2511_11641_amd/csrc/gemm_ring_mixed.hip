// The contraction kernel with one K-slow operand: dY W without a transposed copy of W (with the activation derivatives as
// epilogues), and the combination no layer uses (A K-slow, B K-contiguous), which the contraction entry point offers.
#include "gemm_ring.h"

#define NN_SHAPES(X) X(0, 256, 256, 2) X(4, 256, 128, 3) X(7, 192, 128, 3) X(8, 128, 128, 4) X(9, 64, 128, 4)
#define TN_SHAPES(X) X(0, 256, 256, 2) X(8, 128, 128, 4)
#define NN_INST(I, BM, BN, NS) template __global__ void gemm_bf16_ring_kernel<BM, BN, NS, false, true, false, GEMM_EPIS_NN>(const RingGrid, const GemmDesc);
#define TN_INST(I, BM, BN, NS) template __global__ void gemm_bf16_ring_kernel<BM, BN, NS, true, false, false, GEMM_EPIS_TX>(const RingGrid, const GemmDesc);
NN_SHAPES(NN_INST)
TN_SHAPES(TN_INST)
template __global__ void gemm_bf16_ring_kernel<128, 128, 4, false, true, false, GEMM_EPIS_NN, true>(const RingGrid, const GemmDesc);
template __global__ void gemm_bf16_ring_kernel<128, 128, 4, true, false, false, GEMM_EPIS_TX, true>(const RingGrid, const GemmDesc);

hipError_t gemm_ring_launch_mixed(ecospa_ctx* ctx, const GemmDesc& d, int shape, int k_chunk) {
#define NN_CASE(I, BM, BN, NS) if (shape == I) return ring_launch_shape<BM, BN, NS, false, true, false, GEMM_EPIS_NN>(ctx, d, k_chunk);
#define TN_CASE(I, BM, BN, NS) if (shape == I) return ring_launch_shape<BM, BN, NS, true, false, false, GEMM_EPIS_TX>(ctx, d, k_chunk);
  if (ring_wide(d) && shape == GEMM_RING_WIDE_SHAPE) {
    if (d.trans_b) return ring_launch_shape<128, 128, 4, false, true, false, GEMM_EPIS_NN, true>(ctx, d, k_chunk);
    return ring_launch_shape<128, 128, 4, true, false, false, GEMM_EPIS_TX, true>(ctx, d, k_chunk);
  }
  if (d.trans_b) { NN_SHAPES(NN_CASE) }
  else { TN_SHAPES(TN_CASE) }
  return hipErrorInvalidValue;
}
