// The contraction kernel of resident workgroups for x W^T: the activations that keep their input, and the derivatives (a file of its
// own only to compile in parallel).
#include "gemm_flow.h"

#define FLOW_NT(X) X(EPI_BIAS_ACT) X(EPI_DACT) X(EPI_SWIGLU) X(EPI_DSWIGLU)
#define FLOW_INST(KIND) template __global__ void gemm_bf16_flow_kernel<FLOW_BM, FLOW_BN, FLOW_NS, false, false, KIND, FLOW_NB>(const GemmDesc, int, int);
FLOW_NT(FLOW_INST)

hipError_t gemm_flow_launch_nt_act(ecospa_ctx* ctx, const GemmDesc& d) {
#define FLOW_CASE(KIND) if (d.epi.kind == KIND) return flow_launch<false, false, KIND>(ctx, d);
  FLOW_NT(FLOW_CASE)
  return hipErrorInvalidValue;
}
