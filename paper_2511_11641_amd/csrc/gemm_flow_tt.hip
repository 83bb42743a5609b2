// The contraction kernel of resident workgroups for dY^T X (weight gradients, no column sums).
#include "gemm_flow.h"

template __global__ void gemm_bf16_flow_kernel<FLOW_BM, FLOW_BN, FLOW_NS, true, true, EPI_STORE, FLOW_NB>(const GemmDesc, int, int);

hipError_t gemm_flow_launch_tt(ecospa_ctx* ctx, const GemmDesc& d) {
  if (d.epi.kind != EPI_STORE) return hipErrorInvalidValue;
  return flow_launch<true, true, EPI_STORE>(ctx, d);
}
