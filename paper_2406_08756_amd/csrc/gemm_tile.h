// bf16 matrix products on the CDNA4 matrix cores (v_mfma_f32_32x32x16_bf16).
//
//   C[M, N] = sum_k A(m, k) * B(k, n) (+ bias[n]),   fp32 accumulation
//
// Either operand may be stored "K-major" (the contraction index is the
// contiguous one: activations and weights of a forward linear layer) or
// "MN-major" (the contraction index is the row index: the weight in an input
// gradient, both operands in a weight gradient).
//
// Design.  One workgroup of 8 wavefronts (256 rows per tile; one workgroup per compute unit, see the loop) or of 4 (two
// workgroups per unit) owns a BM x BN output tile, each wavefront a block of it, so every fragment read from LDS feeds
// two to four MFMAs.  K is walked in slabs of 32 or 64.  Slabs travel global memory -> LDS directly (buffer_load_dwordx4
// ... lds, no staging registers and no address arithmetic) through a ring that keeps one to three of them in flight,
// which is what it takes to cover L2 latency at this MFMA rate.  Bank
// conflicts are avoided by permuting 16-byte chunks, applied on the global
// address side since a direct load writes lane i to LDS offset 16 i:
//   K-major slab  [mn][64]: chunk ^= (row >> 1) & 7, [mn][32]: chunk ^= (row >> 2) & 3
//   MN-major slab [k][mn]: chunk ^= (k & 3) << 2 (of 64 columns: ((k >> 1) & 1) << 2), read with the transposing
//     LDS read (ds_read_b64_tr_b16) that hands each lane four consecutive k.
// The product is formed transposed (B fragment as the first MFMA operand) so
// each lane ends with four consecutive n of one row m; the epilogue passes the
// tile through LDS and stores whole rows, 16 bytes per lane.
#pragma once
#include <type_traits>

#include "kernels.h"
#include "mfma_common.h"
#include "pointwise_math.h"
#include "quotient.h"

namespace lynx {
namespace {

constexpr int kStages = 4;     // LDS ring depth in slabs
constexpr int kSlots = 5;      // ... of the 256 x 256 tile of eight wavefronts, in pieces of 32 KB (all of the LDS)

// From this row stride (elements) on, a load's offset from the corner of its tile of up to 256 rows may take more than 32 bits.
constexpr long long kFarStride = 1ll << 22;

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
  // for quotient(): of tiles_m tiles_n, of a band of tile rows (8 tiles_n), of the rows of the last band, and of nz, tiles_n and nz2
  uint32_t inv_tiles, inv_band, inv_last, inv_nz, inv_tiles_n, inv_nz2;
  // split contraction: workgroup x computes K range x / (tiles_m tiles_n) of k_splits ranges of
  // k_per indices (whole slabs; the last range may be shorter, none is empty) and leaves its fp32
  // sums in partial[split][M][N] instead of rounding into C
  int k_splits, k_per;
  float* partial;
  // fused epilogue (GemmEpilogueKind)
  int epi;
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

constexpr int kBand = 8;  // tile rows of a band, see gemm_tile

// Tiles of bm x bn, and the inverses of what their indices are divided by.
inline void set_tiles(MfmaGemmArgs* g, int bm, int bn) {
  g->tiles_m = (g->M + bm - 1) / bm;
  g->tiles_n = (g->N + bn - 1) / bn;
  const long long tiles = static_cast<long long>(g->tiles_m) * g->tiles_n;
  g->inv_tiles = inverse(tiles, tiles * g->k_splits - 1);
  g->inv_band = inverse(static_cast<long long>(kBand) * g->tiles_n, tiles - 1);
  const int last = g->tiles_m % kBand;
  g->inv_last = last != 0 ? inverse(last, static_cast<long long>(last) * g->tiles_n - 1) : 0u;
  g->inv_nz = inverse(g->nz, tiles * g->nz - 1);
  g->inv_tiles_n = inverse(g->tiles_n, tiles - 1);
  g->inv_nz2 = inverse(g->nz2, g->nz - 1);
}

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
//
// FAR: a row stride of kFarStride elements or more.
//
// FORM: a single product, one that carries GeLU (in kernels of its own: with it behind a branch of the epilogue the others
// took 0.2 us longer each, of 7 to 13), or one of a batch of matrices with CausalMode (attention).
enum TileForm { kSingle, kWithGelu, kOfSequence };
template <bool A_KMAJOR, bool B_KMAJOR, int BM, int BN, TileForm FORM, bool SPLITK = false, int STAGES = kStages, bool RAGGED = false,
          int BK = kBK, int WAVES = kWaves, bool SERIAL = false, bool FAR = false>
__device__ __forceinline__ void gemm_tile(const MfmaGemmArgs& g, const int block_x, const int block_z) {
  constexpr bool SEQ = FORM == kOfSequence;
  constexpr int kWavesN = WAVES == 8 ? BN / 64 : 2;
  constexpr int WM = BM * kWavesN / WAVES, WN = BN / kWavesN;  // wavefronts in a grid of WAVES / kWavesN x kWavesN
  constexpr int TM = WM / 32, TN = WN / 32;
  using SA = Slab<BM, A_KMAJOR, BK, WAVES>;
  using SB = Slab<BN, B_KMAJOR, BK, WAVES>;
  constexpr int kStageElems = SA::kElems + SB::kElems;
  constexpr int kLoads = SA::kLoadsPerWave + SB::kLoadsPerWave;  // per wavefront per slab
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* smem = reinterpret_cast<bf16_t*>(smem_raw);

  // workgroup -> output tile
  int tm, tn, bz = block_z, split = 0;
  if (SEQ && (g.causal == kCausalKLeM || g.causal == kCausalKGeM)) {
    // One-dimensional grid over (tile, matrix), longest contraction first: tile row tm
    // contracts over tm + 1 (k <= m) or tiles_m - tm (k >= m) row blocks, and a launch
    // that ends on the long tiles leaves most compute units idle meanwhile.  Matrix z
    // stays on XCD z % 8, whose L2 then keeps its small operand.
    const int t = quotient(block_x, g.nz, g.inv_nz);
    bz = block_x - t * g.nz;
    const int row = quotient(t, g.tiles_n, g.inv_tiles_n);
    tn = t - row * g.tiles_n;
    tm = g.causal == kCausalKLeM ? g.tiles_m - 1 - row : row;
  } else if (SEQ) {
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
    if (SPLITK) {
      split = quotient(block_x, ntiles, g.inv_tiles);
      tile = block_x - split * ntiles;
    }
    const int per_xcd = ntiles / 8;
    if (tile < per_xcd * 8) tile = (tile & 7) * per_xcd + (tile >> 3);
    const int band = quotient(tile, kBand * g.tiles_n, g.inv_band);
    const int in_band = tile - band * kBand * g.tiles_n;
    const int band_rows = min(kBand, g.tiles_m - band * kBand);
    tn = band_rows == kBand ? in_band / kBand : quotient(in_band, band_rows, g.inv_last);
    tm = band * kBand + in_band - tn * band_rows;
  }
  const int m0 = tm * BM, n0 = tn * BN;
  // contraction range: causal products skip the slabs that are identically zero
  int k_begin = 0, k_end = g.K;
  if (SEQ && g.causal == kCausalKLeM) k_end = min(g.K, m0 + BM);
  if (SEQ && g.causal == kCausalKGeM) k_begin = m0;
  if (SPLITK) {
    k_begin = split * g.k_per;
    k_end = min(g.K, k_begin + g.k_per);
  }
  const bf16_t *Abase = g.A, *Bbase = g.B;
  bf16_t* Cbase = g.C;
  if (SEQ) {
    const int z1 = quotient(bz, g.nz2, g.inv_nz2), z2 = bz - z1 * g.nz2;
    Abase += z1 * g.a_z1 + z2 * g.a_z2;
    Bbase += z1 * g.b_z1 + z2 * g.b_z2;
    Cbase += z1 * g.c_z1 + z2 * g.c_z2;
  }

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = wave / kWavesN * WM, wn0 = wave % kWavesN * WN;

  // Where this lane's direct loads of slab 0 start: bytes from the corner of the operand's tile.  (FAR: more than 32
  // bits of them, see kFarStride.)
  using Offset = std::conditional_t<FAR, long long, uint32_t>;
  Offset oa[SA::kLoadsPerWave], ob[SB::kLoadsPerWave];
#pragma unroll
  for (int j = 0; j < SA::kLoadsPerWave; ++j) {
    int mn = SA::lane_mn(wave, j, lane);
    if (RAGGED) mn = min(mn, g.M - m0 - (A_KMAJOR ? 1 : 8));
    const long long k = SA::lane_k(wave, j, lane);
    oa[j] = static_cast<Offset>(2 * (A_KMAJOR ? mn * g.lda + k : k * g.lda + mn));
  }
#pragma unroll
  for (int j = 0; j < SB::kLoadsPerWave; ++j) {
    int mn = SB::lane_mn(wave, j, lane);
    if (RAGGED) mn = min(mn, g.N - n0 - (B_KMAJOR ? 1 : 8));
    const long long k = SB::lane_k(wave, j, lane);
    ob[j] = static_cast<Offset>(2 * (B_KMAJOR ? mn * g.ldb + k : k * g.ldb + mn));
  }
  const char* const corner_a = reinterpret_cast<const char*>(Abase + (A_KMAJOR ? m0 * g.lda + k_begin : k_begin * g.lda + m0));
  const char* const corner_b = reinterpret_cast<const char*>(Bbase + (B_KMAJOR ? n0 * g.ldb + k_begin : k_begin * g.ldb + n0));
  const long long a_step = 2 * (A_KMAJOR ? BK : BK * g.lda);  // bytes per slab
  const long long b_step = 2 * (B_KMAJOR ? BK : BK * g.ldb);

  const int nk = RAGGED ? (k_end - k_begin + BK - 1) / BK : (k_end - k_begin) / BK;
  // the slab that reaches beyond the contraction range (none: -1), and how many of its k exist
  const int k_rem = (k_end - k_begin) % BK;
  const int tail = RAGGED && k_rem != 0 ? nk - 1 : -1;
  const int whole = FAR ? 0 : (tail < 0 ? nk : tail);  // slabs that buffer loads fetch

  // Direct load j of an operand's slab kt to `to` (wavefront-uniform).  Steady: the slab is whole, and the load is a
  // buffer load with the slab's corner in scalar registers, so that no vector instruction goes with it.  (Pointers
  // of 64 bits, advanced in vector registers: 1206 TFLOP/s in the 256 x 256 tile where this gets 1255, and 1083 with
  // the tail's condition on every load.)
  auto load = [&](auto of_b_tag, auto steady_tag, int kt, int j, bf16_t* to) {
    constexpr bool of_b = decltype(of_b_tag)::value;
    const char* corner = of_b ? corner_b + kt * b_step : corner_a + kt * a_step;
    const Offset offset = of_b ? ob[j] : oa[j];
    if constexpr (decltype(steady_tag)::value && !FAR) {
      buffer_load_to_lds(corner, offset, to);
    } else {
      const char* from = corner + offset;
      if (RAGGED && kt == tail && (of_b ? SB::lane_k(wave, j, lane) : SA::lane_k(wave, j, lane)) >= k_rem)
        from = reinterpret_cast<const char*>(&kZeroChunk);
      __builtin_amdgcn_global_load_lds((global_void_ptr)(from), (lds_void_ptr)(to), 16, 0, 0);
    }
  };
  constexpr std::integral_constant<bool, false> kA{}, kAny{};
  constexpr std::integral_constant<bool, true> kB{}, kSteady{};
  // j-th direct load of slab kt (A's first, then B's) -> ring stage kt % STAGES
  auto stage_load = [&](auto steady_tag, int kt, int stage, int j) {
    bf16_t* sa = smem + stage * kStageElems;
    if (j < SA::kLoadsPerWave) load(kA, steady_tag, kt, j, sa + SA::lds_offset(wave, j));
    else load(kB, steady_tag, kt, j - SA::kLoadsPerWave, sa + SA::kElems + SB::lds_offset(wave, j - SA::kLoadsPerWave));
  };
  auto issue_load = [&](auto steady_tag, int kt, int j) { stage_load(steady_tag, kt, kt % STAGES, j); };
  auto issue_slab = [&](auto steady_tag, int kt) {
#pragma unroll
    for (int j = 0; j < kLoads; ++j) issue_load(steady_tag, kt, j);
  };

  // Bias of this wavefront's columns.  Tiles of four wavefronts request it ahead of the contraction (larger ones have no
  // registers to spare and do so in one batch behind it: one exposed round trip to L2).
  constexpr bool kBiasEarly = WAVES == 4 && !SEQ && !SPLITK;
  uint2 braw[TN][4];
  auto request_bias = [&] {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n0 + wn0 + 32 * i + 8 * q + 4 * (lane >> 5);
        braw[i][q] = *reinterpret_cast<const uint2*>(g.bias + (RAGGED ? min(n, g.N - 4) : n));
      }
  };
  if (kBiasEarly && g.bias != nullptr) request_bias();

  floatx16_t acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  if constexpr (WAVES == 8) {
    // Two groups of four wavefronts, one of each per SIMD, take turns: while one multiplies a chunk of 32
    // contraction indices (2 TM TN matrix instructions back to back), the other reads its fragments of the next
    // chunk, and a barrier swaps the roles.  Slabs of 64 indices, whole 128-byte lines of a K-major operand, so two
    // chunks and four phases per slab; every compute phase issues a share of the loads, spread between its matrix
    // instructions (all of a slab's loads in one compute phase: 1104 TFLOP/s where this gets 1255, in a phase
    // that reads fragments 1091).  What bounds it: the clock that the power limit allows, then the issue of the loads.
    //
    // 256 x 256: a ring of five 32 KB slots that A and B slabs take in turn (piece 2 k: A's slab k, piece 2 k + 1:
    // B's); while slab k is multiplied, A(k + 1), B(k + 1) and A(k + 2) are in flight or arriving.  Against eight
    // wavefronts in step on slabs of 32 (ring of four; TFLOP/s, random operands in rotation so that none is cached):
    // 16384 x 2560 x 5120, both K-major 1014 -> 1255; 8192 x 2048 x 8192 1137 -> 1365, with an MN-major B 1252 ->
    // 1365, both MN-major 1252 -> 1364; all-zero operands 1740 -> 2091, 1907 -> 2179, 1827 -> 2153.
    // 256 x 128: whole slabs in a ring of three.
    static_assert(BM == 256 && (BN == 256 || BN == 128) && BK == 64 && !SERIAL, "tiles of eight wavefronts");
    constexpr bool kInTurn = BN == 256;
    static_assert(STAGES == (kInTurn ? kSlots : 3), "ring");
    constexpr int kHalf = kLoads / 2;  // direct loads per wavefront per compute phase
    // load j of the h-th half of a slab's loads (B's and then A's pieces, or A's loads followed by B's), to the
    // ring position `at` (a slot, or a stage)
    auto load_half = [&](auto h_tag, auto steady_tag, int kt, int at, int j) {
      constexpr int h = decltype(h_tag)::value;
      if constexpr (kInTurn) {
        constexpr std::integral_constant<bool, h == 0> of_b{};
        load(of_b, steady_tag, kt, j, smem + at * SA::kElems + SA::lds_offset(wave, j));
      } else {
        const int n = h * kHalf + j;
        if (n < SA::kLoadsPerWave) load(kA, steady_tag, kt, n, smem + at * kStageElems + SA::lds_offset(wave, n));
        else load(kB, steady_tag, kt, n - SA::kLoadsPerWave, smem + at * kStageElems + SA::kElems + SB::lds_offset(wave, n - SA::kLoadsPerWave));
      }
    };
    constexpr std::integral_constant<int, 0> kFirst{};
    constexpr std::integral_constant<int, 1> kSecond{};
    auto load_all = [&](auto h_tag, auto steady_tag, int kt, int at) {
#pragma unroll
      for (int j = 0; j < kHalf; ++j) load_half(h_tag, steady_tag, kt, at, j);
    };
    // The order of halves: in turn, A0 | B0 A1 | B1 A2 | ...: `first half k` is B(k), `second half k` A(k + 1) with
    // its slab counted as k + 1; otherwise the halves of slab k.  `kAhead` slabs after kt, a compute phase of the
    // first group issues half c; the second group, half a slab later in time, has done half 0 a phase before and
    // goes on to the next slab's.  Before the loop: what those phases assume done; then slab 0 has landed.
    auto first_loads = [&](auto steady_tag) {
      constexpr bool steady = decltype(steady_tag)::value;
      if constexpr (kInTurn) {
        load_all(kSecond, steady_tag, 0, 0);
        load_all(kFirst, steady_tag, 0, 1);
        if (steady || nk > 1) {
          load_all(kSecond, steady_tag, 1, 2);
          if (wave >= 4) load_all(kFirst, steady_tag, 1, 3);
        }
      } else {
        load_all(kFirst, steady_tag, 0, 0);
        load_all(kSecond, steady_tag, 0, 0);
        if (steady || nk > 1) {
          load_all(kFirst, steady_tag, 1, 1);
          load_all(kSecond, steady_tag, 1, 1);
          if (wave >= 4 && (steady || nk > 2)) load_all(kFirst, steady_tag, 2, 2);
        }
      }
    };
    if (whole > 2) first_loads(kSteady);
    else first_loads(kAny);
    constexpr int kNewer = kInTurn ? kHalf : 2 * kHalf;  // loads issued after slab kt + 1's when it is waited for
    if (nk > 1) {
      if (wave >= 4 && (kInTurn || nk > 2)) wait_vmcnt<kNewer + kHalf>();
      else wait_vmcnt<kNewer>();
    } else {
      wait_vmcnt<0>();
    }
    block_barrier();
    Frag<A_KMAJOR> fa[2][TM];
    Frag<B_KMAJOR> fb[2][TN];
    // (ragged: a wavefront whose part of the tile lies beyond the output loads and keeps the barriers, no more)
    const bool works = !RAGGED || (m0 + wm0 < g.M && n0 + wn0 < g.N);
    int slot_a = 0, slot_b = 1;  // in turn: of slab kt; otherwise slot_a: its stage
    auto slab_step = [&](const int kt, auto group_tag, auto steady_tag, auto works_tag) {
      constexpr int group = decltype(group_tag)::value;
      constexpr bool steady = decltype(steady_tag)::value;  // no half asked for here is missing or has the tail
      constexpr bool working = decltype(works_tag)::value;
      const bf16_t* sa = smem + slot_a * (kInTurn ? SA::kElems : kStageElems);
      const bf16_t* sb = kInTurn ? smem + slot_b * SA::kElems : sa + SA::kElems;
      // what slab kt - 1 left: its slots, or its stage
      const int free_a = kInTurn ? (slot_a >= 2 ? slot_a - 2 : slot_a - 2 + STAGES) : (slot_a >= 1 ? slot_a - 1 : STAGES - 1);
      const int free_b = slot_b >= 2 ? slot_b - 2 : slot_b - 2 + STAGES;
      // A compute phase's share of loads: which half, of which slab, to where.  Slab kt - 1 was last read one phase
      // before the first group's first compute phase of slab kt, slab kt one before the second group's last.
      constexpr int kHalf0 = kInTurn ? 1 : 2;  // half 0 in the first group's phases of slab kt is slab kt + kHalf0's
      auto issue = [&](auto c_tag, int j) {
        constexpr int c = decltype(c_tag)::value;
        constexpr int h = group == 0 ? c : 1 - c;
        constexpr std::integral_constant<int, h> h_tag{};
        const int of = h == 1 ? kt + 2 : kt + kHalf0 + group;
        const int at = kInTurn ? (group == 0 ? (c == 0 ? free_a : free_b) : (c == 0 ? free_b : slot_a))
                               : (group == 1 && c == 1 ? slot_a : free_a);
        if (steady || of < nk) load_half(h_tag, steady_tag, of, at, j);
      };
      auto chunk = [&](auto c_tag) {
        constexpr int c = decltype(c_tag)::value;
        if (working) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int j = 0; j < TM; ++j) fa[u][j] = SA::fragment(sa, wm0 + 32 * j, 2 * c + u, lane);
#pragma unroll
            for (int i = 0; i < TN; ++i) fb[u][i] = SB::fragment(sb, wn0 + 32 * i, 2 * c + u, lane);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        // Slab kt + 1 has landed, for the first group's next reading phase.  (The first group waits at the
        // end of its compute phase, which is the same phase.)
        if (group == 1 && c == 1) wait_vmcnt<steady ? kNewer : 0>();
        wait_lgkmcnt0();
        if (working) {
#pragma unroll
          for (int u = 0; u < 2; ++u) {
#pragma unroll
            for (int j = 0; j < TM; ++j) fa[u][j].settle();
#pragma unroll
            for (int i = 0; i < TN; ++i) fb[u][i].settle();
          }
        }
        block_barrier</*WAITED=*/true>();
        __builtin_amdgcn_s_setprio(1);
        constexpr int kMfmas = 2 * TM * TN;
        constexpr int kEvery = kMfmas / 4;  // (at most four loads)
#pragma unroll
        for (int m = 0; m < kMfmas; ++m) {
          if (working) {
            // (every second row of blocks backwards, so that each instruction has an operand of the one before it: 0.2 to 0.3 %
            // of a pass of the 1.3B-, 7B- and 13B-shaped layers, whose products run at the clock that the power limit allows;
            // no more than two runs of one build differ by)
            const int u = m / (TM * TN), i = (m / TM) % TN, j = (i & 1) != 0 ? TM - 1 - m % TM : m % TM;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[u][i].operand(), fa[u][j].operand(), acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
          if (m % kEvery == 0 && m / kEvery < kHalf) issue(c_tag, m / kEvery);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (group == 0 && c == 1) wait_vmcnt<steady ? kNewer : 0>();
        block_barrier</*WAITED=*/true>();  // (nothing of this phase is left to issue: see above)
        __builtin_amdgcn_s_setprio(0);
      };
      chunk(kFirst);
      chunk(kSecond);
      if constexpr (kInTurn) {
        slot_a = slot_a + 2 >= STAGES ? slot_a + 2 - STAGES : slot_a + 2;
        slot_b = slot_b + 2 >= STAGES ? slot_b + 2 - STAGES : slot_b + 2;
      } else {
        slot_a = slot_a + 1 == STAGES ? 0 : slot_a + 1;
      }
    };
    // (one phase apart: the second group starts, and the first ends, with a barrier more)
    constexpr int kReach = kInTurn ? 3 : 4;  // a steady step asks for slabs up to kt + kReach - 1, none of them the last
    auto contract = [&](auto group_tag, auto works_tag) {
      if (decltype(group_tag)::value == 1) block_barrier();
      int kt = 0;
      for (; kt + kReach < nk; ++kt) slab_step(kt, group_tag, std::true_type{}, works_tag);
      for (; kt < nk; ++kt) slab_step(kt, group_tag, std::false_type{}, works_tag);
      if (decltype(group_tag)::value == 0) block_barrier();
    };
    if (works) {
      if (wave < 4) contract(kFirst, std::true_type{});
      else contract(kSecond, std::true_type{});
    } else {
      if (wave < 4) contract(kFirst, std::false_type{});
      else contract(kSecond, std::false_type{});
    }
  } else {
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
  if constexpr (A_KMAJOR && B_KMAJOR && TM * TN <= 2) {
    // Little to multiply per slab (four or eight matrix instructions of a wavefront): what counts is the chain from slab
    // to slab.  All fragments of the next slab are requested at once, right behind the barrier that says it has landed, and
    // arrive while this slab's are multiplied; the barrier also frees this slab's stage, whose fragments every
    // wavefront has in registers, so STAGES slabs are in flight.  (With a request and a wait per 16 indices, the loop below, a
    // forward pass of 128 tokens of h 5120 takes 63.6 us where this takes 62.6; with MN-major operands, whose requests are
    // twice as many instructions, that loop is the faster one: small_bf16_store_all 118.8 and 120.3.)
    constexpr int kSteps = BK / 16;
    constexpr int kMfmas = kSteps * TM * TN;
    auto first_slabs = [&](auto steady_tag) {
      constexpr bool steady = decltype(steady_tag)::value;
#pragma unroll
      for (int i = 0; i < STAGES; ++i)
        if (steady || i < nk)
#pragma unroll
          for (int j = 0; j < kLoads; ++j) stage_load(steady_tag, i, i, j);
    };
    if (STAGES <= whole) first_slabs(kSteady);
    else first_slabs(kAny);
    wait_slabs<kLoads, STAGES - 1>(nk - 1);
    block_barrier();
    Frag<A_KMAJOR> fa[2][kSteps][TM];
    Frag<B_KMAJOR> fb[2][kSteps][TN];
    auto request = [&](auto set_tag, int stage) {
      constexpr int set = decltype(set_tag)::value;
      const bf16_t* sa = smem + stage * kStageElems;
#pragma unroll
      for (int u = 0; u < kSteps; ++u) {
#pragma unroll
        for (int j = 0; j < TM; ++j) fa[set][u][j] = SA::fragment(sa, wm0 + 32 * j, u, lane);
#pragma unroll
        for (int i = 0; i < TN; ++i) fb[set][u][i] = SB::fragment(sa + SA::kElems, wn0 + 32 * i, u, lane);
      }
    };
    auto arrived = [&](auto set_tag) {
      constexpr int set = decltype(set_tag)::value;
      wait_lgkmcnt0();
#pragma unroll
      for (int u = 0; u < kSteps; ++u) {
#pragma unroll
        for (int j = 0; j < TM; ++j) fa[set][u][j].settle();
#pragma unroll
        for (int i = 0; i < TN; ++i) fb[set][u][i].settle();
      }
    };
    constexpr std::integral_constant<int, 0> kEven{};
    constexpr std::integral_constant<int, 1> kOdd{};
    request(kEven, 0);
    arrived(kEven);
    int stage = 0;
    auto slab_step = [&](int kt, auto set_tag, auto steady_tag) {
      constexpr int set = decltype(set_tag)::value;
      constexpr bool steady = decltype(steady_tag)::value;
      constexpr std::integral_constant<int, 1 - set> kNext{};
      const int freed = stage;
      stage = stage + 1 == STAGES ? 0 : stage + 1;
      const bool more = steady || kt + 1 < nk;
      if (more) {
        if (steady) wait_vmcnt<(STAGES - 2) * kLoads>();
        else wait_slabs<kLoads, STAGES - 2>(nk - 2 - kt);
        block_barrier</*WAITED=*/true>();
        request(kNext, stage);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int m = 0; m < kMfmas; ++m) {
        const int u = m / (TM * TN), i = m / TM % TN, j = m % TM;
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][u][i].operand(), fa[set][u][j].operand(), acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (m == 0 && (steady || kt + STAGES < nk)) {
#pragma unroll
          for (int j2 = 0; j2 < kLoads; ++j2) stage_load(steady_tag, kt + STAGES, freed, j2);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (more) arrived(kNext);
      end_range(kt);
    };
    int kt = 0;
    for (; kt + 1 + STAGES < whole; kt += 2) {
      slab_step(kt, kEven, std::true_type{});
      slab_step(kt + 1, kOdd, std::true_type{});
    }
    for (; kt < nk; kt += 2) {
      slab_step(kt, kEven, std::false_type{});
      if (kt + 1 < nk) slab_step(kt + 1, kOdd, std::false_type{});
    }
  } else {
  // prologue: STAGES - 1 slabs in flight, the first one landed
  constexpr int kAhead = STAGES - 1;
  static_assert(kAhead >= 1 && (kAhead - 1) * kLoads < 64, "ring depth");
  if (kAhead <= whole) {
#pragma unroll
    for (int i = 0; i < kAhead; ++i) issue_slab(kSteady, i);
  } else {
#pragma unroll
    for (int i = 0; i < kAhead; ++i)
      if (i < nk) issue_slab(kAny, i);
  }
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
            if (refill) issue_load(steady_tag, kt + kAhead, u * kStepLoads + op - TM - TN);
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
  wait_lgkmcnt0();
  settle(0);
  int kt = 0;
  for (; kt + kAhead < whole; ++kt) {
    slab_step(kt, std::true_type{});
    end_range(kt);
  }
  for (; kt < nk; ++kt) {
    slab_step(kt, std::false_type{});
    end_range(kt);
  }
  }
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
  constexpr int kRowChunks = WN / 8;
  constexpr int kRowsPerStore = kWave / kRowChunks;
  constexpr int kIters = WM / kRowsPerStore;
  // (an opaque copy of the lane index: nothing derived from it can be computed, and kept
  // in registers, ahead of the contraction loop)
  int elane = lane;
  asm volatile("" : "+v"(elane));
  const int lr = elane / kRowChunks, lc = elane % kRowChunks;
  const long long row0 = m0 + wm0;
  const int col0 = n0 + wn0, col = col0 + lc * 8;  // first column, this lane's 8 outputs
  // (ragged: what this wavefront may store, relative to its first row and column)
  const int rows_in = RAGGED ? g.M - (m0 + wm0) : WM;
  const bool col_in = !RAGGED || col < g.N;
  // Rows of [M, N] arrays, 16 bytes per lane, this wavefront's block: buffer accesses that end with the block's
  // last row, so rows and columns that do not exist read zeros and are not written, without a branch, and an
  // address is one 32-bit addition.  (With 64-bit products of row and stride, compares and branches per access
  // instead, and two instructions for each three-way exclusive or of the dropout generator: a pass of the 13B-shaped
  // shard, 16384 tokens, 5358 us where this takes 5276, of 8192 tokens of h 1024 1171 and 1151.)
  struct Rows {
    RowBuffer buffer;
    const char* base;      // FAR
    long long stride;      // bytes
    uint32_t first, step;  // this lane's offset in access 0, from one access to the next
  };
  auto rows_of = [&](const bf16_t* p, long long ld) {
    Rows v;
    const bf16_t* corner = p + row0 * ld + col0;
    v.base = reinterpret_cast<const char*>(corner);
    v.stride = 2 * ld;
    if constexpr (!FAR) {
      v.buffer = row_buffer(corner, rows_in > 0 ? static_cast<uint32_t>(min(rows_in, WM)) * static_cast<uint32_t>(2 * ld) : 0u);
      v.first = col_in ? static_cast<uint32_t>(lr) * static_cast<uint32_t>(2 * ld) + 16 * lc : 0x80000000u;
      v.step = static_cast<uint32_t>(kRowsPerStore) * static_cast<uint32_t>(2 * ld);
    }
    return v;
  };
  auto row_load = [&](const Rows& v, int t) {
    if constexpr (FAR) {
      const int r = t * kRowsPerStore + lr;
      uintx4_t x = {0u, 0u, 0u, 0u};
      if (r < rows_in && col_in) x = *reinterpret_cast<const uintx4_t*>(v.base + r * v.stride + 16 * lc);
      return x;
    } else {
      return row_buffer_load(v.buffer, v.first + static_cast<uint32_t>(t) * v.step);
    }
  };
  auto row_store = [&](const Rows& v, int t, uintx4_t x) {
    if constexpr (FAR) {
      const int r = t * kRowsPerStore + lr;
      if (r < rows_in && col_in) *reinterpret_cast<uintx4_t*>(const_cast<char*>(v.base) + r * v.stride + 16 * lc) = x;
    } else {
      row_buffer_store(v.buffer, v.first + static_cast<uint32_t>(t) * v.step, x);
    }
  };
  // Fused epilogues combine every 8 outputs with the same 8 elements of `aux`, fetched in
  // batches of 8 per lane, two batches in flight; the first is requested here, so it
  // arrives while the tile is rounded into LDS.
  constexpr int kBatch = kIters < 8 ? kIters : 8;
  constexpr int kBatches = kIters / kBatch;
  static_assert(kIters % kBatch == 0, "epilogue batches");
  uintx4_t ra0[kBatch], ra1[kBatch];
  const bool fused = FORM != kWithGelu && g.epi != kEpiNone;
  const Rows aux = rows_of(fused ? g.aux : Cbase, fused ? g.aux_ld : g.ldc);
  auto aux_load = [&](uintx4_t (&ra)[kBatch], int batch) {
#pragma unroll
    for (int k = 0; k < kBatch; ++k) ra[k] = row_load(aux, batch * kBatch + k);
  };
  if (fused) aux_load(ra0, 0);
  bf16_t* stage = smem + wave * (WM * WN);
  auto round_to_stage = [&](auto bias_tag) {
    constexpr bool with_bias = decltype(bias_tag)::value;
    if (with_bias && !kBiasEarly) request_bias();
    block_barrier();  // every wavefront is done with the ring (no load is in flight any more)
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nl = 32 * i + 8 * q + 4 * (lane >> 5);
        float bv[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (with_bias) {
          const uint2 b = braw[i][q];
          bv[0] = bf16_lo(b.x); bv[1] = bf16_hi(b.x); bv[2] = bf16_lo(b.y); bv[3] = bf16_hi(b.y);
        }
        auto out = [&](int j, int k) { return with_bias ? acc[i][j][4 * q + k] + bv[k] : acc[i][j][4 * q + k]; };
#pragma unroll
        for (int j = 0; j < TM; ++j) {
          const int ml = 32 * j + (lane & 31);
          uint2 o;
          o.x = pack_bf16(out(j, 0), out(j, 1));
          o.y = pack_bf16(out(j, 2), out(j, 3));
          const int chunk = (nl >> 3) ^ (ml & (kRowChunks - 1));
          *reinterpret_cast<uint2*>(stage + ml * WN + chunk * 8 + (nl & 7)) = o;
        }
      }
  };
  if (g.bias != nullptr) round_to_stage(std::true_type{});
  else round_to_stage(std::false_type{});
  auto staged = [&](int t) {
    const int r = t * kRowsPerStore + lr;
    return *reinterpret_cast<const uintx4_t*>(stage + r * WN + ((lc ^ (r & (kRowChunks - 1))) << 3));
  };
  const Rows out = rows_of(Cbase, g.ldc);
  if (FORM != kWithGelu && !fused) {
#pragma unroll
    for (int t = 0; t < kIters; ++t) row_store(out, t, staged(t));
    return;
  }
  auto unpacked = [](uintx4_t raw, float (&v)[8]) {
    Raw8<bf16_t> r;
    r.v = make_uint4(raw[0], raw[1], raw[2], raw[3]);
    unpack(r, v);
  };
  auto packed = [](const float (&v)[8]) {
    return uintx4_t{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]), pack_bf16(v[4], v[5]), pack_bf16(v[6], v[7])};
  };
  if constexpr (FORM == kWithGelu) {
    // U, where somebody wants it, and G
    const bool keep_u = g.plain != nullptr;
    const Rows plain = rows_of(keep_u ? g.plain : Cbase, g.ldc);
#pragma unroll
    for (int t = 0; t < kIters; ++t) {
      const uintx4_t p = staged(t);
      if (keep_u) row_store(plain, t, p);
      float u[8];
      unpacked(p, u);
#pragma unroll
      for (int i = 0; i < 8; ++i) u[i] = gelu_f(u[i]);
      row_store(out, t, packed(u));
    }
    return;
  }
  auto all_batches = [&](auto&& finish) {
    if (kBatches > 1) aux_load(ra1, 1);
#pragma unroll
    for (int bt = 0; bt < kBatches; bt += 2) {
      finish(ra0, bt);
      if (bt + 2 < kBatches) aux_load(ra0, bt + 2);
      if (bt + 1 < kBatches) {
        finish(ra1, bt + 1);
        if (bt + 3 < kBatches) aux_load(ra1, bt + 3);
      }
    }
  };
  if (g.epi == kEpiBiasDropoutAdd) {
    float bv[8];
    load8(g.vec + (col_in ? col : 0), bv);
    const bool keep_product = g.plain != nullptr;
    const Rows plain = rows_of(keep_product ? g.plain : Cbase, g.ldc);
    // dropout group (8 elements) of access 0, and groups from one access to the next
    const uint64_t group0 = (static_cast<uint64_t>(row0 + lr) * static_cast<uint64_t>(g.N) + col) >> 3;
    const uint64_t groups = static_cast<uint64_t>(kRowsPerStore) * static_cast<uint64_t>(g.N) >> 3;
    all_batches([&](const uintx4_t (&ra)[kBatch], int batch) {
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        const int t = batch * kBatch + k;
        const uintx4_t p = staged(t);
        float prod[8], x[8], o[8];
        unpacked(p, prod);
        unpacked(ra[k], x);
        if (keep_product) row_store(plain, t, p);
        bias_dropout_add8(prod, bv, x, g.key, group0 + static_cast<uint64_t>(t) * groups, o);
        row_store(out, t, packed(o));
      }
    });
    return;
  }
  float colacc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  all_batches([&](const uintx4_t (&ra)[kBatch], int batch) {
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int t = batch * kBatch + k;
      float prod[8], x[8], o[8];
      unpacked(staged(t), prod);
      unpacked(ra[k], x);
      gelu_bwd8<bf16_t>(prod, x, o);
#pragma unroll
      for (int i = 0; i < 8; ++i) colacc[i] += !RAGGED || t * kRowsPerStore + lr < rows_in ? o[i] : 0.f;
      row_store(out, t, packed(o));
    }
  });
  // column sums of this wavefront's WM rows: lanes with the same lc hold different rows
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int o = kRowChunks; o < kWave; o <<= 1) colacc[i] += __shfl_xor(colacc[i], o, kWave);
  if (lane < kRowChunks && rows_in > 0 && col_in) store8(g.colsum_partial + (row0 / WM) * g.N + col, colacc);
}

}  // namespace
}  // namespace lynx
