// Chooses the kernel for a matrix product.
#include "gemm_plans.h"

namespace lynx {
namespace {

bool aligned(const void* p, uintptr_t bytes) { return (reinterpret_cast<uintptr_t>(p) & (bytes - 1)) == 0; }

bool unbatched(const GemmDesc& d) { return d.causal == kCausalNone && d.nz1 * d.nz2 == 1; }

bool gemm_mfma_supported(int dtype, const GemmDesc& d) {
  if (dtype != 1 || d.M % 8 || d.N % 8 || d.K % 8 || d.M <= 0 || d.N <= 0 || d.K <= 0) return false;
  if (d.causal == kCausalOutLower && d.M != d.N) return false;
  if ((d.causal == kCausalKLeM || d.causal == kCausalKGeM) && (d.M != d.K || d.bias != nullptr)) return false;
  if (d.causal == kCausalNone && d.nz1 * d.nz2 != 1) return false;
  const bool a_k = d.a_sk == 1, a_mn = d.a_sm == 1;
  const bool b_k = d.b_sk == 1, b_mn = d.b_sn == 1;
  if (!(a_k || a_mn) || !(b_k || b_mn) || (!a_k && b_k)) return false;
  if ((a_k ? d.a_sm : d.a_sk) % 8 || (b_k ? d.b_sn : d.b_sk) % 8 || d.c_sm % 8) return false;
  if (d.a_sz1 % 8 || d.a_sz2 % 8 || d.b_sz1 % 8 || d.b_sz2 % 8 || d.c_sz1 % 8 || d.c_sz2 % 8) return false;
  if (!aligned(d.A, 16) || !aligned(d.B, 16) || !aligned(d.C, 16) || !aligned(d.bias, 16)) return false;
  switch (d.epi.kind) {
    case kEpiNone:
      return true;
    case kEpiSoftmaxBwd:
      // Only the row-block kernel of the score-shaped products carries it: head dimension 128, whole tiles, at every
      // length.  Elsewhere attn_score_gradient forms the row dot products from the dPd that it differentiates (up to
      // s = 1024), or softmax_dropout_bwd does (beyond); those cancel that tensor's rounding, while these come from the
      // rounded C, which made the error of the QKV weight gradient against 64 bits 0.4 to 2.1 % larger at other shapes.
      // (Up to a size attn_score_gradient_from_c takes these shapes too, with the same dot products.)
      return d.causal == kCausalOutLower && d.bias == nullptr && d.M % 128 == 0 && d.K == 128 && a_k && b_k &&
             d.epi.aux != nullptr && aligned(d.epi.aux, 16) && d.epi.rowdot != nullptr;
    case kEpiBiasDropoutAdd:
      return unbatched(d) && d.bias == nullptr && d.epi.aux != nullptr && aligned(d.epi.aux, 16) &&
             d.epi.aux_ld % 8 == 0 && d.epi.vec != nullptr && aligned(d.epi.vec, 16) && aligned(d.epi.plain, 16);
    case kEpiGelu:
      return unbatched(d) && a_k && b_k && aligned(d.epi.plain, 16);
    case kEpiGeluBwd:  // inside a pair only
      return unbatched(d) && d.bias == nullptr && d.epi.aux != nullptr && aligned(d.epi.aux, 16) &&
             d.epi.aux_ld % 8 == 0 && d.epi.colsum_partial != nullptr && aligned(d.epi.colsum_partial, 16) &&
             d.epi.colsum_out != nullptr;
  }
  return false;
}

}  // namespace

bool gemm_supported(int dtype, const GemmDesc& d) {
  return dtype == 1 ? gemm_mfma_supported(dtype, d) : gemm_f32_supported(d);
}

size_t gemm_scratch_bytes(int dtype, const GemmDesc& d) {
  if (dtype != 1 || !unbatched(d) || d.serial) return 0;
  return ragged_product(d).scratch_bytes;
}

// Tiles of four wavefronts, two workgroups per unit, or a cut contraction's second launch: GeLU costs next to nothing there
// and saves a launch and U's way back, a pass of the fp32 block of 256 tokens of h 256 141.2 -> 138.1 us, of 768 tokens of
// h 512 118.9 -> 116.4, of 984 of h 3016 440.3 -> 433.5, of a drawn small layer 136.8 -> 132.2.  A tile of eight wavefronts has its unit to
// itself, so GeLU adds its 8 us per round to the launch, what the kernel of its own takes: 4000 tokens of h 1600 1206.8
// and 1208.8, 8192 of h 1024 1062.7 and 1062.3, a drawn large layer 1354 and 1373.
bool gemm_absorbs_gelu(int dtype, const GemmDesc& d) {
  if (!gemm_supported(dtype, d)) return false;
  if (dtype != 1) return true;
  const RaggedChoice c = ragged_product(d);
  return c.tile_m <= 128 || c.ranges > 1;
}

hipError_t gemm(int dtype, const GemmDesc& d, float* scratch, size_t scratch_bytes, hipStream_t st) {
  if (!gemm_supported(dtype, d) || d.epi.kind == kEpiGeluBwd) return hipErrorInvalidValue;
  if (d.epi.kind == kEpiGelu && !gemm_absorbs_gelu(dtype, d)) return hipErrorInvalidValue;
  if (dtype != 1) return gemm_f32(d, st);
  if (d.causal != kCausalNone) return gemm_attention(d, st);
  return gemm_ragged(d, scratch, scratch_bytes, st);
}

hipError_t gemm_seq_pair(int dtype, const GemmDesc& first, const GemmDesc& cols, hipStream_t st) {
  if (!gemm_supported(dtype, first) || !gemm_supported(dtype, cols)) return hipErrorInvalidValue;
  if (cols.causal != kCausalKGeM || first.nz1 != cols.nz1 || first.nz2 != cols.nz2) return hipErrorInvalidValue;
  if (dtype != 1) return gemm_f32_two(first, cols, st);
  if (first.causal != kCausalKLeM || first.M != cols.M || first.N != cols.N) return hipErrorInvalidValue;
  return gemm_attention_pair(first, cols, st);
}

bool gemm_pair_supported(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad) {
  if (!gemm_supported(dtype, dgrad) || !gemm_supported(dtype, wgrad)) return false;
  if (!unbatched(dgrad) || !unbatched(wgrad)) return false;
  if (!(dgrad.a_sk == 1 && dgrad.b_sn == 1 && dgrad.b_sk != 1)) return false;  // A K-major, B MN-major
  if (!(wgrad.a_sm == 1 && wgrad.a_sk != 1 && wgrad.b_sn == 1 && wgrad.b_sk != 1)) return false;
  return wgrad.epi.kind == kEpiNone && (dgrad.epi.kind == kEpiNone || dgrad.epi.kind == kEpiGeluBwd);
}

bool gemm_pair_absorbs_gelu(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad) {
  if (!gemm_pair_supported(dtype, dgrad, wgrad)) return false;
  if (dtype != 1) return true;
  // With few rows the plain product is cut into K ranges, which the epilogue's column sums rule out; a
  // GeLU kernel of its own (two launches, three passes over [M, N]) costs less than the product left whole.
  GemmDesc plain = dgrad;
  plain.epi = GemmEpilogue{};
  return ragged_pair(dgrad, wgrad).us <= ragged_pair(plain, wgrad).us + 8.0 + 6.0 * dgrad.M * dgrad.N / 4.0e6;
}

size_t gemm_pair_scratch_bytes(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad) {
  if (dtype != 1) return 0;
  return dgrad.serial ? 0 : ragged_pair(dgrad, wgrad).scratch_bytes;
}

size_t gemm_pair_colsum_bytes(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad) {
  if (dtype != 1) return gemm_f32_pair_colsum_bytes(dgrad, wgrad);
  const int rows = ragged_pair(dgrad, wgrad).colsum_rows;
  return static_cast<size_t>(rows) * static_cast<size_t>(dgrad.N) * sizeof(float);
}

size_t gemm_pair_colsum_least_bytes(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad) {
  if (dtype != 1) return gemm_f32_pair_colsum_bytes(dgrad, wgrad);
  const int cols = (dgrad.N / 8 + 3) / 4 * 8;  // a quarter of the columns, in octets
  return static_cast<size_t>(ragged_pair(dgrad, wgrad).colsum_rows) * static_cast<size_t>(cols) * sizeof(float);
}

hipError_t gemm_pair(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad, float* scratch,
                     size_t scratch_bytes, ColumnSums* sums, hipStream_t st) {
  if (!gemm_pair_supported(dtype, dgrad, wgrad)) return hipErrorInvalidValue;
  if (dtype != 1) return gemm_f32_pair(dgrad, wgrad, nullptr, sums, st);
  return gemm_ragged_pair(dgrad, wgrad, scratch, scratch_bytes, nullptr, sums, st);
}

// In 64 x 64 tiles: layers of which every launch is a hundredth (a pass of 768 tokens of h 512 113.6 -> 112.4 us, of a drawn
// one 132.1 -> 130.0).  Larger tiles keep the launch of its own: with 256 x 256 it gained 0 to 0.4 % of a pass, with
// 128 x 128 it lost 0.3 to 1.2 % (registers), and behind 263 workgroups of 256 x 128, seven more than there are units, the
// launch took 125 us where the two take 107 (larger tiles with the sum last in the launch; between the products not measured).
bool gemm_pair_takes_column_sum(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad) {
  if (!gemm_pair_supported(dtype, dgrad, wgrad)) return false;
  if (dtype != 1) return true;
  const RaggedChoice c = ragged_pair(dgrad, wgrad);
  return c.tile_m == 64 && c.tile_n == 64 && dgrad.epi.kind == kEpiNone && !(dgrad.serial && c.scratch_bytes > 0);
}

hipError_t gemm_pair_column_sum(int dtype, const GemmDesc& dgrad, const GemmDesc& wgrad, float* scratch, size_t scratch_bytes,
                                const ColumnSumInput& in, ColumnSums* sums, hipStream_t st) {
  if (!gemm_pair_takes_column_sum(dtype, dgrad, wgrad) || in.cols % 8) return hipErrorInvalidValue;
  if (dtype != 1) return gemm_f32_pair(dgrad, wgrad, &in, sums, st);
  return gemm_ragged_pair(dgrad, wgrad, scratch, scratch_bytes, &in, sums, st);
}

}  // namespace lynx
