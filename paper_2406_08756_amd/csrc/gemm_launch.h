// What the launchers of the bf16 matrix-core products share.
#pragma once
#include <mutex>

#include "column_partials.h"
#include "dropout_host.h"
#include "gemm_plans.h"
#include "gemm_tile.h"

namespace lynx {

namespace {

// Raises a kernel's dynamic LDS limit, once per call site (i.e. per kernel instantiation) and
// safely when several host threads drive different layers at the same time.
#define LYNX_RAISE_LDS_LIMIT(kern, smem)                                                        \
  do {                                                                                          \
    static std::once_flag once_;                                                                \
    static hipError_t err_ = hipSuccess;                                                        \
    std::call_once(once_, [&] {                                                                 \
      err_ = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),                           \
                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem)); \
    });                                                                                         \
    if (err_ != hipSuccess) return err_;                                                        \
  } while (0)

// Strides that only the tiles with 64-bit load offsets take (kFarStride).
bool is_far(const GemmDesc& d) {
  return (d.a_sk == 1 ? d.a_sm : d.a_sk) >= kFarStride || (d.b_sk == 1 ? d.b_sn : d.b_sk) >= kFarStride ||
         d.c_sm >= kFarStride || (d.epi.kind != kEpiNone && d.epi.aux_ld >= kFarStride);
}

MfmaGemmArgs make_args(const GemmDesc& d) {
  MfmaGemmArgs a{};
  const bool a_k = d.a_sk == 1, b_k = d.b_sk == 1;
  a.A = static_cast<const bf16_t*>(d.A); a.lda = a_k ? d.a_sm : d.a_sk;
  a.B = static_cast<const bf16_t*>(d.B); a.ldb = b_k ? d.b_sn : d.b_sk;
  a.C = static_cast<bf16_t*>(d.C); a.ldc = d.c_sm;
  a.bias = static_cast<const bf16_t*>(d.bias);
  a.M = d.M; a.N = d.N; a.K = d.K;
  a.a_z1 = d.a_sz1; a.a_z2 = d.a_sz2; a.b_z1 = d.b_sz1; a.b_z2 = d.b_sz2;
  a.c_z1 = d.c_sz1; a.c_z2 = d.c_sz2;
  a.nz = d.nz1 * d.nz2; a.nz2 = d.nz2; a.causal = d.causal;
  a.k_splits = 1; a.k_per = d.K; a.partial = nullptr;
  a.epi = d.epi.kind;
  if (d.epi.kind != kEpiNone) {
    a.aux = static_cast<const bf16_t*>(d.epi.aux); a.aux_ld = d.epi.aux_ld;
    a.vec = static_cast<const bf16_t*>(d.epi.vec);
    a.plain = static_cast<bf16_t*>(d.epi.plain);
    a.colsum_partial = d.epi.colsum_partial;
    if (d.epi.kind == kEpiBiasDropoutAdd) a.key = make_dropout_key(d.epi.dp, d.epi.site);
    if (d.epi.kind == kEpiSoftmaxBwd) {
      a.key = make_dropout_key(d.epi.dp, 0);
      a.rowdot = d.epi.rowdot; a.scale = d.epi.scale;
      a.global_heads = d.epi.global_heads; a.head0 = d.epi.head0;
    }
  }
  return a;
}

}  // namespace
}  // namespace lynx
