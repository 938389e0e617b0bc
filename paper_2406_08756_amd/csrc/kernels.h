// Host-callable launchers of the HIP kernels.  Every launcher enqueues on the
// given stream, never synchronises, and returns the launch status.  `dtype`
// is 0 for fp32 storage and 1 for bf16 storage; arithmetic is fp32 throughout.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace lynx {

// Whether a launch of so many workgroups of so many threads is one that HIP takes (fewer than 2^32 threads per dimension).
inline bool fits_grid(long long workgroups, int threads) { return workgroups * threads < (1ll << 32); }

struct DropoutParams {
  uint64_t seed;
  uint64_t step;
  uint32_t layer_id;
  float p;
};

// Index map of the attention-dropout site: element (bi, hd, i, j) of a shard
// has flat index ((bi * global_heads + head0 + hd) * s + i) * s + j.
struct AttnShape {
  int b, a, s;
  int global_heads, head0;
};

// ---- column sums over the rows of a tensor ---------------------------------
// Their first stage runs inside the kernels that form the rows and leaves partial sums, one row of `cols`
// floats per workgroup; the second stage, out[c] = the sum of the partial rows in a fixed order, is asked for
// here and done for every job at once by finish_column_sums (which empties the list).
struct ColumnSums {
  struct Job { const float* part; void* out; int rows, cols; };
  static constexpr int kMaxJobs = 8;
  Job job[kMaxJobs];
  int n = 0;
  hipError_t add(const float* part, void* out, int rows, int cols) {
    if (n == kMaxJobs) return hipErrorInvalidValue;
    job[n++] = {part, out, rows, cols};
    return hipSuccess;
  }
};
hipError_t finish_column_sums(int dtype, ColumnSums* sums, hipStream_t st);

// ---- LayerNorm ------------------------------------------------------------
hipError_t layernorm_fwd(int dtype, const void* x, const void* gamma, const void* beta, void* y,
                         float* mean, float* rstd, int rows, int cols, float eps, hipStream_t st);
// dx_out = dres + dLN/dx (dres may alias nothing; dx_out may alias dres);
// the partial sums of dgamma / dbeta (and dbias) go to `scratch`, their second stage to `sums`.
size_t layernorm_bwd_scratch_bytes(int rows, int cols, bool dropout);
hipError_t layernorm_bwd(int dtype, const void* dy, const void* x, const float* mean,
                         const float* rstd, const void* gamma, const void* dres, void* dx_out,
                         void* dgamma, void* dbeta, float* scratch, int rows, int cols,
                         ColumnSums* sums, hipStream_t st);
// The same, and in the same pass the backward of the bias + dropout + residual operator
// whose output the LayerNorm read: dropped = keep c round(dx_out), dbias = its column sums.
hipError_t layernorm_bwd_dropout_bwd(int dtype, const void* dy, const void* x, const float* mean,
                                     const float* rstd, const void* gamma, const void* dres, void* dx_out,
                                     void* dgamma, void* dbeta, void* dropped, void* dbias, float* scratch,
                                     int rows, int cols, int site, DropoutParams dp, ColumnSums* sums, hipStream_t st);

// ---- attention softmax / dropout -----------------------------------------
// P = softmax_{j<=i}(S * scale) (written if P != null), Pd = keep * P * c
// (written if Pd != null; computed from the storage-rounded P).  Columns
// (i, round_up(i+1, 128)) of every written row are zero-filled.
hipError_t softmax_dropout_fwd(int dtype, const void* S, void* P, void* Pd, AttnShape sh,
                               float scale, DropoutParams dp, hipStream_t st);
// Operators 3 to 5 in one launch (attn_softmax.hip): q and k are [T, a * d] with row stride ld; S, P, Pd as the
// separate kernels leave them, each written if not null.
bool attn_scores_softmax_supported(int dtype, int s, int d, long long ld, long long slices);
hipError_t attn_scores_softmax_fwd(const void* q, const void* k, long long ld, void* S, void* P, void* Pd, AttnShape sh, int d,
                                   float scale, DropoutParams dp, hipStream_t st);
// dS = scale P (dP - sum_j dP P), dP = keep c round(dC V^T), in one launch (s <= 1024): dc [T, a * d] with row stride lddc,
// v with ldv.  With `c` (C, row stride lddc; attn_score_gradient_from_c) the sums come from it, as attn_rowdot forms them.
bool attn_score_gradient_supported(int dtype, int s, int d, long long ld, long long slices);
bool attn_score_gradient_from_c(int dtype, int s, int d, long long ld, long long slices);
hipError_t attn_score_gradient(const void* dc, long long lddc, const void* v, long long ldv, const void* c, const void* P, void* dS,
                               AttnShape sh, int d, float scale, DropoutParams dp, hipStream_t st);
// Pd = keep * P * c from a resident P.
hipError_t attn_dropout_fwd(int dtype, const void* P, void* Pd, AttnShape sh, DropoutParams dp,
                            hipStream_t st);
// dS = scale * P * (dP - sum_j dP * P), dP = keep * dPd * c; dS may alias dPd.
hipError_t softmax_dropout_bwd(int dtype, const void* dPd, const void* P, void* dS, AttnShape sh,
                               float scale, DropoutParams dp, hipStream_t st);

// ---- elementwise over [rows, cols] -----------------------------------------
hipError_t gelu_fwd(int dtype, const void* u, void* g, size_t n, hipStream_t st);
size_t colsum_scratch_bytes(int rows, int cols);
// du = dg * gelu'(u) (du may be dg); dbias[c] = sum_r du[r, c]
hipError_t gelu_bwd(int dtype, const void* dg, const void* u, void* du, void* dbias,
                    float* scratch, int rows, int cols, ColumnSums* sums, hipStream_t st);
// out = res + keep * (in + bias) * c, dropout site `site`, element index r*cols + c
hipError_t bias_dropout_add_fwd(int dtype, const void* in, const void* bias, const void* res,
                                void* out, int rows, int cols, int site, DropoutParams dp,
                                hipStream_t st);
// din = keep * dout * c; dbias[c] = sum_r din[r, c]
hipError_t dropout_bwd(int dtype, const void* dout, void* din, void* dbias, float* scratch,
                       int rows, int cols, int site, DropoutParams dp, ColumnSums* sums, hipStream_t st);
// dbias[c] = sum_r x[r, c]
hipError_t column_sum(int dtype, const void* x, void* dbias, float* scratch, int rows, int cols,
                      ColumnSums* sums, hipStream_t st);
// out[(bi * a + hd) * s + i] = sum_dd x[t, hd * d + dd] * y[t, hd * d + dd], t = bi * s + i (fp32);
// x and y are [T, a * d] with row stride ld.  With x = dC and y = C this is the row dot
// product sum_j dP_ij P_ij of the softmax backward.
hipError_t attn_rowdot(int dtype, const void* x, const void* y, float* out, int b, int a, int s, int d,
                       long long ld, hipStream_t st);
// ---- attention without the seq x seq tensors (attn_fused.hip) ----------------------------
// bf16 storage, head dimension 128, sequence a multiple of 128.
bool attn_fused_supported(int dtype, int s, int d);
size_t attn_fused_stats_bytes(int b, int a, int s);
// Operators 3-6 in one launch: C [T, a * d] (row stride ldc) from QKV [T, 3 a d] (row stride
// ld), bit-identical to S -> softmax -> dropout -> Pd V run one after the other; also leaves
// per row (b, head, i) the maximum of the logits and the reciprocal of the row sum in
// stats [b * a * s][2], from which the backward kernels rebuild P.
hipError_t attn_fused_fwd(const void* qkv, long long ld, void* c, long long ldc, float* stats, AttnShape sh, int d,
                          float scale, DropoutParams dp, hipStream_t st);

// Backward of operators 6-4 without P and Pd.  First kernel: dS [b, a, s, s] (dense layout,
// j <= i defined) = scale P (keep c round(dC V^T) - rowdot), P rebuilt from QKV and stats.
// Second kernel: the v block of dqkv [T, 3 a d] = Pd^T dC, Pd rebuilt likewise.  Both
// bit-identical to the unfused kernels run on stored P and Pd.
hipError_t attn_fused_bwd_ds(const void* qkv, long long ld, const void* dc, long long lddc, const float* stats,
                             const float* rowdot, void* ds, AttnShape sh, int d, float scale, DropoutParams dp,
                             hipStream_t st);
hipError_t attn_fused_bwd_dv(const void* qkv, long long ld, const void* dc, long long lddc, const float* stats,
                             void* dqkv, long long lddq, AttnShape sh, int d, float scale, DropoutParams dp,
                             hipStream_t st);

// keep-mask bytes for parity checks: n elements starting at flat index 0 of
// site 1/2, or the [b, a, s, s] tensor of site 0.
hipError_t dropout_mask_hidden(uint8_t* out, size_t n, int site, DropoutParams dp, hipStream_t st);
hipError_t dropout_mask_attn(uint8_t* out, AttnShape sh, DropoutParams dp, hipStream_t st);

// ---- matrix products ------------------------------------------------------
enum CausalMode : int {
  kCausalNone = 0,
  kCausalOutLower = 1,  // only outputs with n <= m are needed (others may be skipped)
  kCausalKLeM = 2,      // contraction restricted to k <= m
  kCausalKGeM = 3       // contraction restricted to k >= m
};

// Elementwise work a matrix-core product can absorb into the pass that stores its output
// tile, so the operator that would read the product back never runs as a kernel of its
// own.  P = the product rounded to storage, exactly what an unfused launch would store.
enum GemmEpilogueKind : int {
  kEpiNone = 0,
  // bias + dropout + residual (operators 8, 13): C = aux + keep (P + vec) c at dropout site
  // `site`, element index m * N + n; if `plain` is not null P is stored there as well (row
  // stride = c_sm).  Bit-identical to bias_dropout_add_fwd run on a stored P.
  kEpiBiasDropoutAdd = 1,
  // GeLU backward (input gradient of FC2 only, inside gemm_pair): C = P gelu'(aux) and
  // colsum_out[n] = sum_m C[m, n] (the FC1 bias gradient): partial sums to `colsum_partial`, second stage to the
  // pair's `sums`.  With room for gemm_pair_colsum_bytes (`colsum_bytes`) in one launch; with less (at least
  // gemm_pair_colsum_least_bytes) in ranges of columns, each with both of its stages before the next: the same bits.
  kEpiGeluBwd = 2,
  // GeLU (operators 10 + 11): U = the product with its bias, rounded, is stored to `plain` unless that is null, and C =
  // gelu(U).  Bit-identical to gelu_fwd run on a stored U.
  kEpiGelu = 3,
  // dropout + softmax backward (B5 + B4) on the score-shaped product dPd = dC V^T (causal,
  // batched): C = dS = scale aux (keep c P - rowdot), aux = the softmax output P in the layout
  // of C, rowdot[z * M + i] the row's sum_j dP_ij P_ij (attn_rowdot), dropout site 0 with the
  // attention index map (global_heads, head0).  dPd itself is never stored.
  kEpiSoftmaxBwd = 4
};
struct GemmEpilogue {
  int kind;
  const void* aux;        // [M, N], row stride aux_ld: the residual (1) or U (2)
  long long aux_ld;
  const void* vec;        // (1) bias[N]
  void* plain;            // (1) (3) nullable
  int site;               // (1)
  DropoutParams dp;       // (1)
  float* colsum_partial;  // (2)
  size_t colsum_bytes;    // (2)
  void* colsum_out;       // (2) [N], storage dtype
  const float* rowdot;    // (4)
  float scale;            // (4)
  int global_heads, head0;  // (4)
};

// C[z][m, n] = sum_k A[z][m, k] * B[z][k, n] (+ bias[n]), z = (z1, z2) a
// two-level batch.  Element strides are explicit, so any operand may be a
// transposed or column-sliced view.  Accumulation is fp32 in a fixed order.
struct GemmDesc {
  int M, N, K;
  const void* A; long long a_sm, a_sk, a_sz1, a_sz2;
  const void* B; long long b_sk, b_sn, b_sz1, b_sz2;
  void* C; long long c_sm, c_sz1, c_sz2;  // C is row-major within a matrix (n stride 1)
  const void* bias;                        // nullable, length N, same dtype
  int nz1, nz2;
  int causal;                              // CausalMode
  GemmEpilogue epi;                        // kind 0 (none) unless the matrix-core path is used
  // No room for the partial sums of a contraction that is cut for speed: one workgroup sums its ranges one after
  // the other (slower, same bits).  In a pair, of both products.
  bool serial;
};
// Picks a kernel.  `scratch` (fp32, 16-byte aligned, gemm_scratch_bytes or more; null when that is 0)
// takes the partial sums of a contraction that is cut into ranges; they are added in a fixed order.
hipError_t gemm(int dtype, const GemmDesc& d, float* scratch, size_t scratch_bytes, hipStream_t st);
size_t gemm_scratch_bytes(int dtype, const GemmDesc& d);  // shapes and `serial` only
// Sizes multiples of 8, operands 16-byte aligned and contiguous along one index, an epilogue this
// product can carry: everything the layer asks for except fp32 with kEpiSoftmaxBwd.
bool gemm_supported(int dtype, const GemmDesc& d);
// Two products that do not need each other in one launch: C = sq y (kCausalKLeM) and C' = sq^T y' (kCausalKGeM) over the
// same seq x seq operand (dQ and dK from dS); fp32 also a score-shaped product (kCausalOutLower) in the place of the first
// (dPd and dV).  bf16: the bits of gemm() on each.  fp32: the tile, and with it whether a contraction is one sum or four,
// is chosen for both together.
hipError_t gemm_seq_pair(int dtype, const GemmDesc& first, const GemmDesc& cols, hipStream_t st);
// Whether a forward product should carry GeLU (kEpiGelu): supported, and it pays.
bool gemm_absorbs_gelu(int dtype, const GemmDesc& d);
// Input gradient and weight gradient of one linear layer in one launch.  `scratch` as above
// (gemm_pair_scratch_bytes).
hipError_t gemm_pair(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad, float* scratch,
                     size_t scratch_bytes, ColumnSums* sums, hipStream_t st);
// The same, and the column sums of x [rows, cols] in the same launch, where gemm_pair_takes_column_sum: partial sums to `part`
// (not part of `scratch`), second stage to `sums`.  The bits of column_sum.
struct ColumnSumInput {
  const void* x;
  void* out;
  float* part;
  int rows, cols;
};
hipError_t gemm_pair_column_sum(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad, float* scratch, size_t scratch_bytes,
                                const ColumnSumInput& in, ColumnSums* sums, hipStream_t st);
bool gemm_pair_takes_column_sum(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad);
size_t gemm_pair_scratch_bytes(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad);  // shapes, epilogue and `serial` only
// Whether the input gradient should carry the GeLU backward (kEpiGeluBwd): supported, and it pays.
bool gemm_pair_absorbs_gelu(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad);
size_t gemm_pair_colsum_bytes(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad);  // its column partials
size_t gemm_pair_colsum_least_bytes(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad);

}  // namespace lynx
