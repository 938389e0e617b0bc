// Which form of a kernel would run, answered on the host, so that a test that means to reach a form can say so and fail
// when it no longer does.  Exported, but not part of the C ABI that lynx.h declares.
#include "gemm_plans.h"

extern "C" {

// Attention of bf16 layers, with row stride ld of QKV; bits: 1, operators 3 to 5
// in one launch; 2, the score gradient in one launch that keeps dPd in registers; 4, dQ and dK in one launch.
unsigned lynx_form_attention(int s, int d, long long ld, int batch, int heads) {
  using namespace lynx;
  const long long slices = static_cast<long long>(batch) * heads;
  GemmDesc rows{};
  rows.M = s; rows.N = d; rows.K = s;
  rows.a_sm = s; rows.a_sk = 1;
  rows.b_sk = ld; rows.b_sn = 1;
  rows.c_sm = ld;
  rows.nz1 = batch; rows.nz2 = heads;
  rows.causal = kCausalKLeM;
  return (attn_scores_softmax_supported(1, s, d, ld, slices) ? 1u : 0u) | (attn_score_gradient_supported(1, s, d, ld, slices) ? 2u : 0u) |
         (gemm_attention_pair_joint(rows) ? 4u : 0u);
}

}  // extern "C"
