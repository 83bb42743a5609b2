// A weight gradient on 192 x 128 tiles together with an x W^T (a file per shape only to compile in parallel).
#include "gemm_ring.h"

#define PAIR_NT(X) X(4, 256, 128, 3) X(5, 192, 192, 3) X(7, 192, 128, 3) X(8, 128, 128, 4)
#define PAIR_INST(I, BM, BN, NS)                                                                                          \
  template __global__ void gemm_bf16_pair_kernel<192, 128, 3, false, BM, BN, NS>(const RingGrid, const RingGrid, int, const GemmDesc, const GemmDesc); \
  template __global__ void gemm_bf16_pair_kernel<192, 128, 3, true, BM, BN, NS>(const RingGrid, const RingGrid, int, const GemmDesc, const GemmDesc);
PAIR_NT(PAIR_INST)

hipError_t gemm_pair_launch_192(ecospa_ctx* ctx, const GemmDesc& w, const GemmDesc& x, int x_shape, int w_k_chunk) {
#define PAIR_CASE(I, BM, BN, NS)                                                                                          \
  if (x_shape == I) return w.colsum ? ring_launch_pair<192, 128, 3, true, BM, BN, NS>(ctx, w, x, w_k_chunk)              \
                                    : ring_launch_pair<192, 128, 3, false, BM, BN, NS>(ctx, w, x, w_k_chunk);
  PAIR_NT(PAIR_CASE)
  return hipErrorInvalidValue;
}
