// The matrix-core products behind gemm() and gemm_pair(): which kernels there are, and what the
// choice between them needs to know.  Host only.
#pragma once
#include "kernels.h"

namespace lynx {

// What the ragged kernels would do with a product (or a pair): estimated time, fp32 scratch for the
// partial sums of cut contractions, (pair) rows of column partials of the GeLU epilogue, the tile, and the ranges that
// the contraction (pair: of the weight gradient, of the input gradient) is cut into.
struct RaggedChoice {
  double us;
  size_t scratch_bytes;
  int colsum_rows;
  int tile_m, tile_n;
  int ranges, dgrad_ranges;
};
RaggedChoice ragged_product(const GemmDesc& d);
RaggedChoice ragged_pair(const GemmDesc& dgrad, const GemmDesc& wgrad);
hipError_t gemm_ragged(const GemmDesc& d, float* scratch, size_t scratch_bytes, hipStream_t st);
// (with a column sum, nullable: gemm_pair_column_sum)
hipError_t gemm_ragged_pair(const GemmDesc& dgrad, const GemmDesc& wgrad, float* scratch, size_t scratch_bytes,
                            const ColumnSumInput* in, ColumnSums* sums, hipStream_t st);
// Products of attention (gemm_mfma.hip).
hipError_t gemm_attention(const GemmDesc& d, hipStream_t st);
int attention_score_run(int s, int slices);  // score-shaped ones: tiles per workgroup
// ... and (gemm_ragged.hip) a product over the rows and one over the columns of the same seq x seq operand in one launch.
// (two where one would have more threads than a launch may)
hipError_t gemm_attention_pair(const GemmDesc& rows, const GemmDesc& cols, hipStream_t st);
bool gemm_attention_pair_joint(const GemmDesc& rows);

// fp32 storage (gemm_f32.hip).
bool gemm_f32_supported(const GemmDesc& d);
struct F32Choice { int tile, stages; };  // side of the tile, ring stages
F32Choice gemm_f32_choice(const GemmDesc& d);
F32Choice gemm_f32_pair_choice(const GemmDesc& dgrad, const GemmDesc& wgrad);
hipError_t gemm_f32(const GemmDesc& d, hipStream_t st);
// two products of attention, the second with both operands MN-major, in one launch
hipError_t gemm_f32_two(const GemmDesc& a, const GemmDesc& b, hipStream_t st);
size_t gemm_f32_pair_colsum_bytes(const GemmDesc& dgrad, const GemmDesc& wgrad);
hipError_t gemm_f32_pair(const GemmDesc& dgrad, const GemmDesc& wgrad, const ColumnSumInput* in, ColumnSums* sums, hipStream_t st);

}  // namespace lynx
