// bf16 matrix products on the CDNA4 matrix cores (v_mfma_f32_32x32x16_bf16).
//
//   C[M, N] = sum_k A(m, k) * B(k, n) (+ bias[n]),   fp32 accumulation
//
// Either operand may be stored "K-major" (the contraction index is the
// contiguous one: activations and weights of a forward linear layer) or
// "MN-major" (the contraction index is the row index: the weight in an input
// gradient, both operands in a weight gradient).
//
// Design.  One workgroup of 4 wavefronts (one per SIMD, up to 512 registers
// each) owns a BM x BN output tile (256 x 256 when it divides); each
// wavefront owns a quarter of it, so every fragment read from LDS feeds four
// MFMAs.  K is walked in slabs of 32.  Slabs travel global memory -> LDS
// directly (global_load_lds_dwordx4, no staging registers) through a ring of
// four LDS stages: while one slab is multiplied, three more are in flight,
// which is what it takes to cover L2 latency at this MFMA rate.  Bank
// conflicts are avoided by permuting 16-byte chunks, applied on the global
// address side since a direct load writes lane i to LDS offset 16 i:
//   K-major slab  [mn][32]: chunk ^= (row >> 2) & 3
//   MN-major slab [32][mn]: chunk ^= (k & 3) << 2, read with the transposing
//     LDS read (ds_read_b64_tr_b16) that hands each lane four consecutive k.
// The product is formed transposed (B fragment as the first MFMA operand) so
// each lane ends with four consecutive n of one row m; the epilogue passes the
// tile through LDS and stores whole rows, 16 bytes per lane.
#pragma once
#include <type_traits>

#include "kernels.h"
#include "mfma_common.h"
#include "pointwise_math.h"

namespace lynx {
namespace {

constexpr int kStages = 4;     // LDS ring depth

struct MfmaGemmArgs {
  const bf16_t* A; long long lda;
  const bf16_t* B; long long ldb;
  bf16_t* C; long long ldc;
  const bf16_t* bias;
  int M, N, K;
  int tiles_m, tiles_n;
  // batched use (attention): matrix z = z1 * nz2 + z2 starts at these element offsets
  long long a_z1, a_z2, b_z1, b_z2, c_z1, c_z2;
  int nz, nz2;
  int causal;  // CausalMode
  int run;     // score-shaped row-block kernels: tiles per workgroup
  // split contraction: workgroup x computes K range x / (tiles_m tiles_n) of k_splits ranges of
  // k_per indices (whole slabs; the last range may be shorter, none is empty) and leaves its fp32
  // sums in partial[split][M][N] instead of rounding into C
  int k_splits, k_per;
  float* partial;
  // fused epilogue (GemmEpilogueKind).  aux / vec / plain are indexed with the absolute
  // column col0 + n, so a launch that covers a column range of the output (edge strips)
  // passes them unchanged; row_len is the full row length (the dropout element index).
  int epi;
  int col0, row_len;
  const bf16_t* aux; long long aux_ld;
  const bf16_t* vec;
  bf16_t* plain;
  float* colsum_partial;
  DropoutKey key;
  // kEpiSoftmaxBwd (attention): per-row dot products, 1 / sqrt(d), dropout index map
  const float* rowdot;
  float scale;
  int global_heads, head0;
};

// 16 bytes of zeros: what a ragged tile multiplies in place of contraction indices beyond K.
__device__ const uint4 kZeroChunk = {0u, 0u, 0u, 0u};

// One output tile: `block_x` selects the tile, `block_z` the matrix of a batch.
//
// RAGGED: M, N and K need not be whole tiles, only multiples of 8 (every dimension of this library
// is).  Rows and 8-column chunks beyond the operand repeat its last ones, so every address is inside
// it, and their outputs are not stored; contraction indices beyond K, which only the last slab can
// have, read zeros.  Nothing else differs, so a tile that is whole has the bits of the plain form.
//
// SERIAL: the K ranges (k_per indices, whole slabs) of a cut contraction one after the other: each is summed
// from zero and added to the sum of those before it, which is what SPLITK and the launch that adds its partial
// sums do, bit for bit, with registers in the place of the partial sums.
template <bool A_KMAJOR, bool B_KMAJOR, int BM, int BN, bool SPLITK = false, int STAGES = kStages, bool RAGGED = false,
          int BK = kBK, int WAVES = kWaves, bool SERIAL = false>
__device__ __forceinline__ void gemm_tile(const MfmaGemmArgs& g, const int block_x, const int block_z) {
  constexpr int kWavesN = WAVES / 2;
  constexpr int WM = BM / 2, WN = BN / kWavesN;  // wavefronts in a grid of 2 x kWavesN
  constexpr int TM = WM / 32, TN = WN / 32;
  using SA = Slab<BM, A_KMAJOR, BK, WAVES>;
  using SB = Slab<BN, B_KMAJOR, BK, WAVES>;
  constexpr int kStageElems = SA::kElems + SB::kElems;
  constexpr int kLoads = SA::kLoadsPerWave + SB::kLoadsPerWave;  // per wavefront per slab
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* smem = reinterpret_cast<bf16_t*>(smem_raw);

  // workgroup -> output tile
  int tm, tn, bz = block_z;
  if (g.causal == kCausalKLeM || g.causal == kCausalKGeM) {
    // One-dimensional grid over (tile, matrix), longest contraction first: tile row tm
    // contracts over tm + 1 (k <= m) or tiles_m - tm (k >= m) row blocks, and a launch
    // that ends on the long tiles leaves most compute units idle meanwhile.  Matrix z
    // stays on XCD z % 8, whose L2 then keeps its small operand.
    const int t = block_x / g.nz;
    bz = block_x - t * g.nz;
    const int row = t / g.tiles_n;
    tn = t - row * g.tiles_n;
    tm = g.causal == kCausalKLeM ? g.tiles_m - 1 - row : row;
  } else if (g.causal == kCausalOutLower) {
    // square output, only tiles on or below the diagonal: t = tm (tm + 1) / 2 + tn
    const int t = block_x;
    tm = static_cast<int>((sqrtf(8.0f * static_cast<float>(t) + 1.0f) - 1.0f) * 0.5f);
    while (tm * (tm + 1) / 2 > t) --tm;
    while ((tm + 1) * (tm + 2) / 2 <= t) ++tm;
    tn = t - tm * (tm + 1) / 2;
  } else {
    // Consecutive workgroup ids land on different XCDs (round robin over 8), so give
    // each XCD a contiguous run of tiles, ordered in bands of 8 tile-rows so a band's
    // panels stay in that XCD's L2.
    const int ntiles = g.tiles_m * g.tiles_n;
    int tile = block_x;
    if (SPLITK) tile = block_x % ntiles;
    const int per_xcd = ntiles / 8;
    if (tile < per_xcd * 8) tile = (tile & 7) * per_xcd + (tile >> 3);
    constexpr int kBand = 8;
    const int band = tile / (kBand * g.tiles_n);
    const int band_rows = min(kBand, g.tiles_m - band * kBand);
    const int in_band = tile - band * kBand * g.tiles_n;
    tm = band * kBand + in_band % band_rows;
    tn = in_band / band_rows;
  }
  const int m0 = tm * BM, n0 = tn * BN;
  // contraction range: causal products skip the slabs that are identically zero
  int k_begin = 0, k_end = g.K;
  if (g.causal == kCausalKLeM) k_end = min(g.K, m0 + BM);
  if (g.causal == kCausalKGeM) k_begin = m0;
  const int split = SPLITK ? block_x / (g.tiles_m * g.tiles_n) : 0;
  if (SPLITK) {
    k_begin = split * g.k_per;
    k_end = min(g.K, k_begin + g.k_per);
  }
  const int z1 = bz / g.nz2, z2 = bz - z1 * g.nz2;
  const bf16_t* Abase = g.A + z1 * g.a_z1 + z2 * g.a_z2;
  const bf16_t* Bbase = g.B + z1 * g.b_z1 + z2 * g.b_z2;
  bf16_t* Cbase = g.C + z1 * g.c_z1 + z2 * g.c_z2;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = wave / kWavesN * WM, wn0 = wave % kWavesN * WN;

  // this lane's global source of each direct load, at slab 0
  const bf16_t* ga[SA::kLoadsPerWave];
  const bf16_t* gb[SB::kLoadsPerWave];
#pragma unroll
  for (int j = 0; j < SA::kLoadsPerWave; ++j) {
    long long mn = m0 + SA::lane_mn(wave, j, lane);
    const long long k = k_begin + SA::lane_k(wave, j, lane);
    if (RAGGED) mn = min(mn, static_cast<long long>(g.M - (A_KMAJOR ? 1 : 8)));
    ga[j] = Abase + (A_KMAJOR ? mn * g.lda + k : k * g.lda + mn);
  }
#pragma unroll
  for (int j = 0; j < SB::kLoadsPerWave; ++j) {
    long long mn = n0 + SB::lane_mn(wave, j, lane);
    const long long k = k_begin + SB::lane_k(wave, j, lane);
    if (RAGGED) mn = min(mn, static_cast<long long>(g.N - (B_KMAJOR ? 1 : 8)));
    gb[j] = Bbase + (B_KMAJOR ? mn * g.ldb + k : k * g.ldb + mn);
  }
  const long long a_step = A_KMAJOR ? BK : BK * g.lda;  // elements per slab
  const long long b_step = B_KMAJOR ? BK : BK * g.ldb;

  const int nk = RAGGED ? (k_end - k_begin + BK - 1) / BK : (k_end - k_begin) / BK;
  // the slab that reaches beyond the contraction range (none: -1), and how many of its k exist
  const int k_rem = (k_end - k_begin) % BK;
  const int tail = RAGGED && k_rem != 0 ? nk - 1 : -1;

  // j-th direct load of slab kt (A pieces first, then B) -> ring stage kt % STAGES
  auto issue_load = [&](int kt, int j) {
    bf16_t* sa = smem + (kt % STAGES) * kStageElems;
    if (j < SA::kLoadsPerWave) {
      const bf16_t* from = ga[j] + kt * a_step;
      if (RAGGED && kt == tail && SA::lane_k(wave, j, lane) >= k_rem) from = reinterpret_cast<const bf16_t*>(&kZeroChunk);
      __builtin_amdgcn_global_load_lds((global_void_ptr)(from),
                                       (lds_void_ptr)(sa + SA::lds_offset(wave, j)), 16, 0, 0);
    } else {
      const int jb = j - SA::kLoadsPerWave;
      const bf16_t* from = gb[jb] + kt * b_step;
      if (RAGGED && kt == tail && SB::lane_k(wave, jb, lane) >= k_rem) from = reinterpret_cast<const bf16_t*>(&kZeroChunk);
      __builtin_amdgcn_global_load_lds((global_void_ptr)(from),
                                       (lds_void_ptr)(sa + SA::kElems + SB::lds_offset(wave, jb)), 16,
                                       0, 0);
    }
  };
  auto issue_slab = [&](int kt) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) issue_load(kt, j);
  };

  floatx16_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  // prologue: STAGES - 1 slabs in flight, the first one landed
  constexpr int kAhead = STAGES - 1;
  static_assert(kAhead >= 1 && (kAhead - 1) * kLoads < 64, "ring depth");
#pragma unroll
  for (int i = 0; i < kAhead; ++i)
    if (i < nk) issue_slab(i);
  wait_slabs<kLoads, kAhead - 1>(nk - 1);
  block_barrier();

  // Two sets of fragments: step u of a slab multiplies set u % 2 while the other set is read.
  Frag<A_KMAJOR> fa[2][TM];
  Frag<B_KMAJOR> fb[2][TN];
  auto settle = [&](int set) {
#pragma unroll
    for (int j = 0; j < TM; ++j) fa[set][j].settle();
#pragma unroll
    for (int i = 0; i < TN; ++i) fb[set][i].settle();
  };
#pragma unroll
  for (int j = 0; j < TM; ++j) fa[0][j] = SA::fragment(smem, wm0 + 32 * j, 0, lane);
#pragma unroll
  for (int i = 0; i < TN; ++i) fb[0][i] = SB::fragment(smem + SA::kElems, wn0 + 32 * i, 0, lane);

  // One slab = BK / 16 steps of TM x TN MFMAs.  The side work is spread between the MFMAs
  // so the matrix pipe never waits for an issue burst: each step but the last reads the
  // fragments of the next one and issues its share of the loads that refill the ring stage
  // every wavefront finished before the last barrier; then [next slab landed?] [barrier];
  // during the last step the next slab's first fragments are read.  `steady` = STAGES - 1 more
  // slabs exist, so the refill and the waits need no conditions.
  constexpr int kSteps = BK / 16;
  constexpr int kMfmas = TM * TN;
  constexpr int kStepLoads = (kLoads + kSteps - 2) / (kSteps - 1);  // refill loads per step
  constexpr int kSide = TM + TN + kStepLoads;                       // side operations of a step
  constexpr int kPer = (kSide + kMfmas - 1) / kMfmas;               // per MFMA
  constexpr int kPerLast = (TM + TN + kMfmas - 1) / kMfmas;
  auto slab_step = [&](int kt, auto steady_tag) {
    constexpr bool steady = decltype(steady_tag)::value;
    const bf16_t* sa = smem + (kt % STAGES) * kStageElems;
    const bf16_t* sb = sa + SA::kElems;
    const bool refill = steady || kt + kAhead < nk;
#pragma unroll
    for (int u = 0; u < kSteps - 1; ++u) {
      const int cur = u & 1, nxt = cur ^ 1;
#pragma unroll
      for (int m = 0; m < kMfmas; ++m) {
        const int i = m / TM, j = m % TM;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cur][i].operand(), fa[cur][j].operand(), acc[i][j], 0, 0, 0);
#pragma unroll
        for (int v = 0; v < kPer; ++v) {
          const int op = m * kPer + v;
          if (op < TM) fa[nxt][op] = SA::fragment(sa, wm0 + 32 * op, u + 1, lane);
          else if (op < TM + TN) fb[nxt][op - TM] = SB::fragment(sb, wn0 + 32 * (op - TM), u + 1, lane);
          else if (op < kSide && u * kStepLoads + op - TM - TN < kLoads) {
            if (refill) issue_load(kt + kAhead, u * kStepLoads + op - TM - TN);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (u < kSteps - 2) {
        wait_lgkmcnt0();
        settle(nxt);
      }
    }
    // the next slab must have landed (newer ones may still be in flight), and all
    // of this wavefront's reads of the current slab must be complete
    if (steady) wait_vmcnt<(kAhead - 1) * kLoads>();
    else wait_slabs<kLoads, kAhead - 1>(nk - 2 - kt);
    wait_lgkmcnt0();
    block_barrier</*WAITED=*/true>();
    constexpr int last = (kSteps - 1) & 1;
    settle(last);
    const bool more = steady || kt + 1 < nk;
    const bf16_t* na = smem + ((kt + 1) % STAGES) * kStageElems;
    const bf16_t* nb = na + SA::kElems;
#pragma unroll
    for (int m = 0; m < kMfmas; ++m) {
      const int i = m / TM, j = m % TM;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[last][i].operand(), fa[last][j].operand(), acc[i][j], 0, 0, 0);
#pragma unroll
      for (int v = 0; v < kPerLast; ++v) {
        const int op = m * kPerLast + v;
        if (more) {
          if (op < TM) fa[last ^ 1][op] = SA::fragment(na, wm0 + 32 * op, 0, lane);
          else if (op < TM + TN) fb[last ^ 1][op - TM] = SB::fragment(nb, wn0 + 32 * (op - TM), 0, lane);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_lgkmcnt0();  // the next slab's first fragments have arrived
    if (more) settle(last ^ 1);
  };
  static_assert(!(SERIAL && SPLITK), "ranges one after the other, or one each");
  floatx16_t total[SERIAL ? TN : 1][SERIAL ? TM : 1];  // SERIAL: sum of the ranges that are complete
  if constexpr (SERIAL) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) total[i][j][r] = -0.f;  // (-0 + x has the bits of x)
  }
  const int range_slabs = SERIAL ? g.k_per / BK : 0;
  auto end_range = [&](int kt) {
    if constexpr (SERIAL) {
      if (kt + 1 < nk && (kt + 1) % range_slabs != 0) return;
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            total[i][j][r] += acc[i][j][r];
            acc[i][j][r] = kt + 1 < nk ? 0.f : total[i][j][r];
          }
    }
  };
  wait_lgkmcnt0();
  settle(0);
  int kt = 0;
  for (; kt + kAhead < (tail < 0 ? nk : tail); ++kt) {
    slab_step(kt, std::true_type{});
    end_range(kt);
  }
  for (; kt < nk; ++kt) {
    slab_step(kt, std::false_type{});
    end_range(kt);
  }

  // Epilogue.  acc[i][j][r] is the element n = wn0 + 32 i + 8 (r/4) + 4 (lane/32) + r%4,
  // m = wm0 + 32 j + lane%32.  Each wavefront rounds its quarter tile (+ bias) to bf16 into
  // its own region of the now idle LDS ring and writes it out as whole rows, 16 bytes per
  // lane.  16-byte chunks of LDS row r are XORed with r so both the 8-byte writes and the
  // 16-byte row reads spread over all banks.
  if (SPLITK) {
    // partial sums of one K range: fp32, four consecutive n per lane
    float* pw = g.partial + (static_cast<long long>(split) * g.M + m0 + wm0 + (lane & 31)) * g.N + n0 + wn0 +
                4 * (lane >> 5);
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float4 v = {acc[i][j][4 * q + 0], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2],
                            acc[i][j][4 * q + 3]};
          if (!RAGGED || (m0 + wm0 + 32 * j + (lane & 31) < g.M && n0 + wn0 + 32 * i + 8 * q + 4 * (lane >> 5) < g.N))
            *reinterpret_cast<float4*>(pw + static_cast<long long>(32 * j) * g.N + 32 * i + 8 * q) = v;
        }
    return;
  }
  // The bias values of this wavefront's columns, requested in one batch (one exposed L2
  // round trip instead of one per group of columns).
  uint2 braw[TN][4];
  if (g.bias != nullptr) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
      {
        const int n = n0 + wn0 + 32 * i + 8 * q + 4 * (lane >> 5);
        braw[i][q] = *reinterpret_cast<const uint2*>(g.bias + (RAGGED ? min(n, g.N - 4) : n));
      }
  }
  constexpr int kRowChunks = WN / 8;
  constexpr int kRowsPerStore = kWave / kRowChunks;
  constexpr int kIters = WM / kRowsPerStore;
  // (an opaque copy of the lane index: nothing derived from it can be computed, and kept
  // in registers, ahead of the contraction loop)
  int elane = lane;
  asm volatile("" : "+v"(elane));
  const int lr = elane / kRowChunks, lc = elane % kRowChunks;
  const long long row0 = m0 + wm0;
  const int col = g.col0 + n0 + wn0 + lc * 8;  // absolute column of this lane's 8 outputs
  // (ragged: what this wavefront may store, relative to its first row and column)
  const int rows_in = RAGGED ? g.M - (m0 + wm0) : WM;
  const bool col_in = !RAGGED || n0 + wn0 + lc * 8 < g.N;
  auto stores = [&](int r) { return !RAGGED || (r < rows_in && col_in); };
  // Fused epilogues combine every 8 outputs with the same 8 elements of `aux`, fetched in
  // batches of 8 per lane, two batches in flight; the first is requested here, so it
  // arrives while the tile is rounded into LDS.
  constexpr int kBatch = kIters < 8 ? kIters : 8;
  constexpr int kBatches = kIters / kBatch;
  static_assert(kIters % kBatch == 0, "epilogue batches");
  uintx4_t ra0[kBatch], ra1[kBatch];
  const bf16_t* auxp = g.epi != kEpiNone ? g.aux + row0 * g.aux_ld + (col_in ? col : g.col0) : nullptr;
  auto aux_load = [&](uintx4_t (&ra)[kBatch], int batch) {
#pragma unroll
    for (int k = 0; k < kBatch; ++k)
    {
      const int r = (batch * kBatch + k) * kRowsPerStore + lr;
      // (ragged: row rows_in - 1 of this wavefront, negative if it has none, is the last row of the operand)
      ra[k] = *reinterpret_cast<const uintx4_t*>(auxp + static_cast<long long>(RAGGED ? min(r, rows_in - 1) : r) * g.aux_ld);
    }
  };
  if (g.epi != kEpiNone) aux_load(ra0, 0);
  block_barrier();  // every wavefront is done with the ring (no load is in flight any more)
  bf16_t* stage = smem + wave * (WM * WN);
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int nl = 32 * i + 8 * q + 4 * (lane >> 5);
      float bv[4] = {0.f, 0.f, 0.f, 0.f};
      if (g.bias != nullptr) {
        const uint2 b = braw[i][q];
        bv[0] = bf16_lo(b.x); bv[1] = bf16_hi(b.x); bv[2] = bf16_lo(b.y); bv[3] = bf16_hi(b.y);
      }
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int ml = 32 * j + (lane & 31);
        uint2 o;
        o.x = pack_bf16(acc[i][j][4 * q + 0] + bv[0], acc[i][j][4 * q + 1] + bv[1]);
        o.y = pack_bf16(acc[i][j][4 * q + 2] + bv[2], acc[i][j][4 * q + 3] + bv[3]);
        const int chunk = (nl >> 3) ^ (ml & (kRowChunks - 1));
        *reinterpret_cast<uint2*>(stage + ml * WN + chunk * 8 + (nl & 7)) = o;
      }
    }
  bf16_t* cw = Cbase + static_cast<long long>(m0 + wm0) * g.ldc + n0 + wn0;
  if (g.epi == kEpiNone) {
#pragma unroll
    for (int t = 0; t < kIters; ++t) {
      const int r = t * kRowsPerStore + lr;
      const uint4 v = *reinterpret_cast<const uint4*>(stage + r * WN + ((lc ^ (r & (kRowChunks - 1))) << 3));
      if (stores(r)) *reinterpret_cast<uint4*>(cw + static_cast<long long>(r) * g.ldc + lc * 8) = v;
    }
    return;
  }
  float bv[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (g.epi == kEpiBiasDropoutAdd) load8(g.vec + (col_in ? col : g.col0), bv);
  float colacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto finish = [&](const uintx4_t (&ra)[kBatch], int batch) {
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int r = (batch * kBatch + k) * kRowsPerStore + lr;
      Raw8<bf16_t> pv, xv;
      pv.v = *reinterpret_cast<const uint4*>(stage + r * WN + ((lc ^ (r & (kRowChunks - 1))) << 3));
      xv.v = make_uint4(ra[k][0], ra[k][1], ra[k][2], ra[k][3]);
      float prod[8], x[8], o[8];
      unpack(pv, prod);
      unpack(xv, x);
      if (g.epi == kEpiBiasDropoutAdd) {
        if (g.plain != nullptr && stores(r))
          *reinterpret_cast<uint4*>(g.plain + (row0 + r) * g.ldc + col) = pv.v;
        const uint64_t elem = static_cast<uint64_t>(row0 + r) * static_cast<uint64_t>(g.row_len) + col;
        bias_dropout_add8(prod, bv, x, g.key, elem >> 3, o);
      } else {
        gelu_bwd8<bf16_t>(prod, x, o);
#pragma unroll
        for (int i = 0; i < 8; ++i) colacc[i] += !RAGGED || r < rows_in ? o[i] : 0.f;
      }
      if (stores(r)) store8(cw + static_cast<long long>(r) * g.ldc + lc * 8, o);
    }
  };
  if (kBatches > 1) aux_load(ra1, 1);
  for (int bt = 0; bt < kBatches; bt += 2) {
    finish(ra0, bt);
    if (bt + 2 < kBatches) aux_load(ra0, bt + 2);
    if (bt + 1 < kBatches) {
      finish(ra1, bt + 1);
      if (bt + 3 < kBatches) aux_load(ra1, bt + 3);
    }
  }
  if (g.epi == kEpiGeluBwd) {
    // column sums of this wavefront's WM rows: lanes with the same lc hold different rows
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int o = kRowChunks; o < kWave; o <<= 1) colacc[i] += __shfl_xor(colacc[i], o, kWave);
    if (lane < kRowChunks && stores(0))
      store8(g.colsum_partial + (row0 / WM) * g.row_len + col, colacc);
  }
}

}  // namespace
}  // namespace lynx
