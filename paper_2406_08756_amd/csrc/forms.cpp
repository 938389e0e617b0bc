// Which form of a kernel would run, answered on the host, so that a test that means to reach a form can say so and fail
// when it no longer does.  Exported, but not part of the C ABI that lynx.h declares.
#include "gemm_plans.h"
#include "quotient.h"

extern "C" {

// Attention of bf16 layers, with row stride ld of QKV; bits: 1, operators 3 to 5
// in one launch; 2, the score gradient in one launch that keeps dPd in registers; 4, dQ and dK in one launch; 8, the score
// gradient in one launch with its row sums from C.
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
         (gemm_attention_pair_joint(rows) ? 4u : 0u) | (attn_score_gradient_from_c(1, s, d, ld, slices) ? 8u : 0u);
}

// x / d as the kernels form it, for x up to `most`, and whether by the inverse.
int lynx_form_quotient(int x, int d, long long most, int* by_inverse) {
  const uint32_t inv = lynx::inverse(d, most);
  *by_inverse = inv != 0;
  return lynx::quotient(x, d, inv);
}

// Tiles per workgroup of the score-shaped products (S where it is formed alone, dPd).
int lynx_form_score_run(int s, int slices) { return lynx::attention_score_run(s, slices); }

// The bf16 product [M, N] over K of a forward linear layer: {rows and columns of the tile, ranges of the contraction}.
void lynx_form_product(int M, int N, int K, int* out) {
  lynx::GemmDesc d{};
  d.M = M; d.N = N; d.K = K;
  const lynx::RaggedChoice c = lynx::ragged_product(d);
  out[0] = c.tile_m; out[1] = c.tile_n; out[2] = c.ranges;
}

// Both bf16 gradients of a linear layer of `inputs` to `outputs`: {rows and columns of the tile, ranges of the weight
// gradient's contraction, of the input gradient's, whether that one carries the GeLU backward}, which `gelu` (FC2) asks
// for where it pays.
void lynx_form_pair(int tokens, int outputs, int inputs, int gelu, int* out) {
  void* const some = reinterpret_cast<void*>(256);  // (aligned; nothing is read)
  lynx::GemmDesc d{}, w{};
  d.M = tokens; d.N = inputs; d.K = outputs;
  d.a_sm = outputs; d.a_sk = 1;
  d.b_sk = inputs; d.b_sn = 1;
  w.M = outputs; w.N = inputs; w.K = tokens;
  w.a_sm = 1; w.a_sk = outputs;
  w.b_sk = inputs; w.b_sn = 1;
  for (lynx::GemmDesc* g : {&d, &w}) {
    g->A = g->B = some;
    g->C = some;
    g->c_sm = inputs;
    g->nz1 = g->nz2 = 1;
  }
  if (gelu) {
    d.epi.kind = lynx::kEpiGeluBwd;
    d.epi.aux = some;
    d.epi.aux_ld = inputs;
    d.epi.colsum_partial = static_cast<float*>(some);
    d.epi.colsum_out = some;
    if (!lynx::gemm_pair_absorbs_gelu(1, d, w)) d.epi = lynx::GemmEpilogue{};
  }
  const lynx::RaggedChoice c = lynx::ragged_pair(d, w);
  out[0] = c.tile_m; out[1] = c.tile_n; out[2] = c.ranges; out[3] = c.dgrad_ranges;
  out[4] = d.epi.kind == lynx::kEpiGeluBwd;
}

// fp32, a linear layer of `inputs` to `outputs`: {side of the tile, ring stages} of the forward product, of the pair of gradients.
void lynx_form_f32(int tokens, int outputs, int inputs, int* out) {
  lynx::GemmDesc f{}, d{}, w{};
  f.M = tokens; f.N = outputs; f.K = inputs;
  d.M = tokens; d.N = inputs; d.K = outputs;
  w.M = outputs; w.N = inputs; w.K = tokens;
  for (lynx::GemmDesc* g : {&f, &d, &w}) g->nz1 = g->nz2 = 1;
  const lynx::F32Choice of_f = lynx::gemm_f32_choice(f), of_pair = lynx::gemm_f32_pair_choice(d, w);
  out[0] = of_f.tile; out[1] = of_f.stages;
  out[2] = of_pair.tile; out[3] = of_pair.stages;
}

}  // extern "C"
