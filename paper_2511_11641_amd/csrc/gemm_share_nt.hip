// x W^T of few tokens, K shared out over the wavefronts of a workgroup.
#include "gemm_share.h"

#define SHARE_SHAPES(X) X(0, 32, 16, 8, 3) X(1, 32, 32, 8, 2) X(2, 64, 16, 8, 2) X(3, 64, 32, 4, 3)
#define SHARE_INST(I, BM, BN, W, D) template __global__ void gemm_bf16_share_kernel<BM, BN, W, D>(const RingGrid, const GemmDesc);
SHARE_SHAPES(SHARE_INST)

hipError_t gemm_share_launch_nt(ecospa_ctx* ctx, const GemmDesc& d, int shape) {
#define SHARE_CASE(I, BM, BN, W, D) if (shape == I) return share_launch_shape<BM, BN, W, D>(ctx, d);
  SHARE_SHAPES(SHARE_CASE)
  return hipErrorInvalidValue;
}
