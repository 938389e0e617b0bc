// bf16 products of linear layers, any size: tiles from 256 x 256 down to 64 x 64, each able to overhang the
// operands, and contractions cut into ranges whose fp32 partial sums a second launch adds in a fixed order.
// plan_product / plan_pair_ragged choose by a cost model.
#include <mutex>

#include "dropout_host.h"
#include "gemm_launch.h"

namespace lynx {
namespace {

// The tiles.  The two largest: eight wavefronts in two groups that take turns (gemm_tile.h).  256 x 128 reads 1.5 times
// as much per operation but gives twice the workgroups: 8192 x 1024 x 4096 1086 TFLOP/s against 876 with
// 256 x 256 (128 workgroups) and 980 with 128 x 128; before these had this form 641, 796 and 980.
// The others: four wavefronts, two workgroups per compute unit.  BK and ring depth: one barrier per 64 contraction
// indices pays where a slab is so little work that the barrier and the LDS round trip dominate it (64 x 64, K = 4096,
// one workgroup: 26.8 us with slabs of 32, 19.0 with 64) and where both operands are K-major, whose rows
// then arrive as whole 128-byte lines (128 x 128 at 4096^3: 182 -> 151 us); with an MN-major operand
// the deeper ring of slabs of 32 is the faster one (128 x 128 at 4096^3: 148 against 150, 146 against 153).
enum RaggedTile { kT256 = 0, kT256x128, kT128, kT128x64, kT64, kNumRaggedTiles };
template <int TILE, bool BOTH_KMAJOR> struct TileShape;
template <bool B> struct TileShape<kT256, B> { static constexpr int BM = 256, BN = 256, BK = 64, S = kSlots, share = 1, waves = 8; };
template <bool B> struct TileShape<kT256x128, B> { static constexpr int BM = 256, BN = 128, BK = 64, S = 3, share = 1, waves = 8; };
template <> struct TileShape<kT128, true> { static constexpr int BM = 128, BN = 128, BK = 64, S = 2, share = 2, waves = 4; };
template <> struct TileShape<kT128, false> { static constexpr int BM = 128, BN = 128, BK = 32, S = 4, share = 2, waves = 4; };
template <bool B> struct TileShape<kT128x64, B> { static constexpr int BM = 128, BN = 64, BK = 64, S = 3, share = 2, waves = 4; };
template <bool B> struct TileShape<kT64, B> { static constexpr int BM = 64, BN = 64, BK = 64, S = 4, share = 2, waves = 4; };

// LDS: S slabs of both operands, or (256 x 256) S slots of one slab each
template <typename T> constexpr size_t tile_lds =
    static_cast<size_t>(T::S) * (T::BN == 256 ? T::BM : T::BM + T::BN) * T::BK * sizeof(bf16_t);
// rows of a wavefront's part of a tile: one row of the GeLU epilogue's column partials
constexpr int kTileWaveRows[kNumRaggedTiles] = {128, 64, 64, 64, 32};
template <int TILE> constexpr int tile_threads = TileShape<TILE, false>::waves * kWave;
template <int TILE> constexpr int tile_waves_per_simd = TileShape<TILE, false>::share * TileShape<TILE, false>::waves / 4;

// Time of 32 contraction indices of a tile, in us: one workgroup on an otherwise idle chip; one on every
// compute unit; `share` on every unit (then for all of them together).  `fixed`: what a round of
// workgroups takes beside its contraction.
//
// The numbers are fitted to measurements, for forward products and for gradient pairs each: 589 products
// and 582 pairs of layers with 64 to 16384 tokens and widths from 40 to 22000, every tile and nearly every cut
// of each timed on operands in rotation, the constants chosen so that the tile and cut with the least predicted time
// lose as little as possible against the fastest: 0.8 % and 2.0 % on average.  What decides no choice is not pinned by
// that: single constants are no times of anything (pairs of 64 x 64 tiles: 0.112 alone, 0.081 with one on every unit), and
// they say little beyond those sizes.  None of the products had an epilogue, nor had the pairs: the store pass with bias,
// dropout and residual is not in the model, and for those the choice is that of the plain product; neither is the GeLU
// pass (984 tokens of h 3016, f 1544: 51 us in 64 x 64 tiles, 47 in the 128 x 128 ones of the model before; of 60 layers'
// FC2 gradients the one that got slower with this model, the others 1.00 to 2.45 times as fast, 1.13 on average).  The
// fit is older than what the K-major tiles of four wavefronts do now (a third of the instructions ahead of the first loads, a slab's fragments
// requested at once, GeLU in FC1's store pass) and was not repeated for them.
struct TileCost {
  int bm, bn, share;
  double alone, one_each, full;
  double fixed;
  // us per 32 indices of a round of n workgroups (n <= kUnits * share)
  double slab(double n) const {
    if (n <= kUnits) return alone + (one_each - alone) * n / kUnits;
    return one_each + (full - one_each) * (n - kUnits) / (kUnits * (share - 1));
  }
  static constexpr int kUnits = 256;  // compute units
};
constexpr TileCost kProductCost[kNumRaggedTiles] = {
    {256, 256, 1, 0.469, 0.603, 0.603, 6.9}, {256, 128, 1, 0.289, 0.381, 0.381, 5.6}, {128, 128, 2, 0.262, 0.402, 0.477, 4.0},
    {128, 64, 2, 0.090, 0.263, 0.290, 4.1}, {64, 64, 2, 0.095, 0.101, 0.616, 4.0}};
constexpr TileCost kPairCost[kNumRaggedTiles] = {
    {256, 256, 1, 0.609, 0.611, 0.611, 4.4}, {256, 128, 1, 0.124, 0.416, 0.416, 8.3}, {128, 128, 2, 0.247, 0.253, 0.478, 4.4},
    {128, 64, 2, 0.172, 0.228, 0.538, 4.1}, {64, 64, 2, 0.112, 0.081, 0.219, 3.2}};
// the launch that adds the partial sums of a cut contraction (product / pair)
constexpr double kFinishFixed[2] = {3.6, 2.7}, kFinishBytesPerUs[2] = {3.4e6, 1.9e6};

constexpr int kMaxBK = 64;   // K ranges of a cut contraction are whole slabs of every tile
constexpr int kCuts[] = {1, 2, 3, 4, 6, 8, 12, 16};   // K ranges considered
constexpr int kMinRange = 256;                        // ... of at least this many indices

int ceil_div(int a, int b) { return (a + b - 1) / b; }
// Indices per range when K is cut into at most `want` ranges of whole slabs (of every tile).
int range_of(int K, int want) { return ceil_div(K, kMaxBK * want) * kMaxBK; }

// us of a launch of one product: rounds of `share` workgroups on every unit
double product_cost(const TileCost& t, int M, int N, int K, int k_per) {
  const int splits = ceil_div(K, k_per);
  const double slabs = static_cast<double>(ceil_div(k_per < K ? k_per : K, 32));
  long long wgs = static_cast<long long>(ceil_div(M, t.bm)) * ceil_div(N, t.bn) * splits;
  const long long round = static_cast<long long>(TileCost::kUnits) * t.share;
  const long long whole = wgs / round;
  wgs -= whole * round;
  double us = static_cast<double>(whole) * (t.fixed + slabs * t.full);
  if (wgs > 0) us += t.fixed + slabs * t.slab(static_cast<double>(wgs));
  if (splits > 1) us += kFinishFixed[0] + (static_cast<double>(splits) * 4 * M * N) / kFinishBytesPerUs[0];
  return us;
}

struct ProductPlan {
  int tile, k_per;
  double us;
  int splits(int K) const { return ceil_div(K, k_per); }
};

ProductPlan search_product(int M, int N, int K) {
  ProductPlan best{kT64, range_of(K, 1), 1e30};
  const bool far = K >= kFarStride || N >= kFarStride;  // the row strides
  for (int t = far ? kT64 : 0; t < kNumRaggedTiles; ++t)
    for (int want : kCuts) {
      if (want > 1 && K < kMinRange * want) break;
      const int k_per = range_of(K, want);
      const double us = product_cost(kProductCost[t], M, N, K, k_per);
      if (us < best.us) best = {t, k_per, us};
    }
  return best;
}

// A plan is a function of the shape alone; a layer asks for the same few again and again, so every
// thread keeps the last ones it worked out.
template <typename Plan, int KEYS>
struct PlanCache {
  static constexpr int kSlots = 256;  // (with 32, the products of one layer in six fell on one another)
  struct Entry { int key[KEYS]; Plan plan; bool used; } entry[kSlots] = {};
  template <typename F>
  const Plan& get(const int (&key)[KEYS], F&& search) {
    unsigned h = 0;
    for (int k : key) h = (h ^ static_cast<unsigned>(k)) * 0x9E3779B1u;
    Entry& e = entry[(h >> 16) % kSlots];
    bool same = e.used;
    for (int i = 0; i < KEYS; ++i) same = same && e.key[i] == key[i];
    if (!same) {
      e.plan = search();
      for (int i = 0; i < KEYS; ++i) e.key[i] = key[i];
      e.used = true;
    }
    return e.plan;
  }
};

ProductPlan plan_product(const GemmDesc& d) {
  static thread_local PlanCache<ProductPlan, 3> cache;
  return cache.get({d.M, d.N, d.K}, [&] { return search_product(d.M, d.N, d.K); });
}

// ---- kernels ------------------------------------------------------------------
template <bool AK, bool BK_, int TILE, bool FAR, TileForm FORM>
__global__ void __launch_bounds__((tile_threads<TILE>), (tile_waves_per_simd<TILE>))
gemm_ragged_kernel(MfmaGemmArgs g) {
  using T = TileShape<TILE, AK && BK_>;
  if (FORM == kSingle && g.k_splits > 1) gemm_tile<AK, BK_, T::BM, T::BN, kSingle, true, T::S, true, T::BK, T::waves, false, FAR>(g, blockIdx.x, 0);
  else gemm_tile<AK, BK_, T::BM, T::BN, FORM, false, T::S, true, T::BK, T::waves, false, FAR>(g, blockIdx.x, FORM == kOfSequence ? blockIdx.y : 0);
}

// Both products of a linear layer's backward in one launch: the first n_first workgroups belong to the one
// whose tiles take longer, the others behind them fill what they leave idle.  (Weight gradient first
// throughout: 237 us for 4000 tokens, 1600 inputs and 6400 outputs, whose input gradient has the longer
// contraction; 198 this way.)
template <int TILE, bool FAR>
__device__ __forceinline__ void pair_tile(const MfmaGemmArgs& wgrad, const MfmaGemmArgs& dgrad, int n_first, int dgrad_first, int x) {
  using T = TileShape<TILE, false>;
  // the second product starts at a multiple of 8 workgroups, as its tile order, which takes the workgroup
  // id mod 8 for the XCD, needs it; the few workgroups in between idle
  const int n_pad = (n_first + 7) & ~7;
  if (x >= n_first && x < n_pad) return;
  const int tile = x < n_first ? x : x - n_pad;
  if ((x < n_first) != (dgrad_first != 0)) {
    if (wgrad.k_splits > 1) gemm_tile<false, false, T::BM, T::BN, kSingle, true, T::S, true, T::BK, T::waves, false, FAR>(wgrad, tile, 0);
    else gemm_tile<false, false, T::BM, T::BN, kSingle, false, T::S, true, T::BK, T::waves, false, FAR>(wgrad, tile, 0);
  } else {
    if (dgrad.k_splits > 1) gemm_tile<true, false, T::BM, T::BN, kSingle, true, T::S, true, T::BK, T::waves, false, FAR>(dgrad, tile, 0);
    else gemm_tile<true, false, T::BM, T::BN, kSingle, false, T::S, true, T::BK, T::waves, false, FAR>(dgrad, tile, 0);
  }
}
template <int TILE, bool FAR>
__global__ void __launch_bounds__((tile_threads<TILE>), (tile_waves_per_simd<TILE>))
gemm_ragged_pair_kernel(MfmaGemmArgs wgrad, MfmaGemmArgs dgrad, int n_first, int dgrad_first) {
  pair_tile<TILE, FAR>(wgrad, dgrad, n_first, dgrad_first, blockIdx.x);
}
// ... and a column sum besides, in workgroups between them
template <int TILE, bool FAR>
__global__ void __launch_bounds__((tile_threads<TILE>), (tile_waves_per_simd<TILE>))
gemm_ragged_pair_guest_kernel(MfmaGemmArgs wgrad, MfmaGemmArgs dgrad, int n_first, int dgrad_first, ColumnPartials guest) {
  const int x = static_cast<int>(blockIdx.x);
  if (x >= guest.first && x < guest.end)
    column_partials<bf16_t>(guest, (x - guest.first) * TileShape<TILE, false>::waves + static_cast<int>(threadIdx.x) / kWave);
  else
    pair_tile<TILE, FAR>(wgrad, dgrad, n_first, dgrad_first, x < guest.first ? x : x - (guest.end - guest.first));
}

template <bool AK, bool BK_, int TILE, bool FAR, TileForm FORM>
hipError_t launch_ragged(MfmaGemmArgs a, hipStream_t st) {
  using T = TileShape<TILE, AK && BK_>;
  constexpr size_t smem = tile_lds<T>;
  auto kern = gemm_ragged_kernel<AK, BK_, TILE, FAR, FORM>;
  LYNX_RAISE_LDS_LIMIT(kern, smem);
  set_tiles(&a, T::BM, T::BN);
  const int ntiles = a.causal == kCausalOutLower ? a.tiles_m * (a.tiles_m + 1) / 2 : a.tiles_m * a.tiles_n * a.k_splits;
  const bool flat = a.causal == kCausalKLeM || a.causal == kCausalKGeM;  // (tile, matrix) in x
  hipLaunchKernelGGL(kern, flat ? dim3(ntiles * a.nz) : dim3(ntiles, a.nz), dim3(T::waves * kWave), smem, st, a);
  return hipGetLastError();
}

template <bool AK, bool BK_>
hipError_t launch_tile(int tile, bool far, const MfmaGemmArgs& a, hipStream_t st) {
  if (a.causal != kCausalNone) {  // attention, in tiles of at most 128 x 128
    if (far) return launch_ragged<AK, BK_, kT64, true, kOfSequence>(a, st);
    switch (tile) {
      case kT128: return launch_ragged<AK, BK_, kT128, false, kOfSequence>(a, st);
      case kT128x64: return launch_ragged<AK, BK_, kT128x64, false, kOfSequence>(a, st);
      default: return launch_ragged<AK, BK_, kT64, false, kOfSequence>(a, st);
    }
  }
  if constexpr (AK && BK_) {  // GeLU in the store pass, in tiles of four wavefronts
    if (a.epi == kEpiGelu && a.k_splits == 1) {
      if (far) return launch_ragged<AK, BK_, kT64, true, kWithGelu>(a, st);
      switch (tile) {
        case kT128: return launch_ragged<AK, BK_, kT128, false, kWithGelu>(a, st);
        case kT128x64: return launch_ragged<AK, BK_, kT128x64, false, kWithGelu>(a, st);
        case kT64: return launch_ragged<AK, BK_, kT64, false, kWithGelu>(a, st);
        default: return hipErrorInvalidValue;
      }
    }
  }
  if (far) return launch_ragged<AK, BK_, kT64, true, kSingle>(a, st);
  if constexpr (AK) {  // (no larger one for two MN-major operands)
    if (tile == kT256) return launch_ragged<AK, BK_, kT256, false, kSingle>(a, st);
    if (tile == kT256x128) return launch_ragged<AK, BK_, kT256x128, false, kSingle>(a, st);
  }
  switch (tile) {
    case kT128: return launch_ragged<AK, BK_, kT128, false, kSingle>(a, st);
    case kT128x64: return launch_ragged<AK, BK_, kT128x64, false, kSingle>(a, st);
    default: return launch_ragged<AK, BK_, kT64, false, kSingle>(a, st);
  }
}

// The ranges of a cut contraction in one workgroup, one after the other (GemmDesc::serial).  The smallest tile,
// whichever the plan has: a product is cut because its tiles are few, and the tile does not enter the sums.
// Latency of the whole contraction on a part of the chip bounds it; it is for workspaces that have no room for the
// cut form.  128 tokens of h 5120 (QKV of width 1920, FC1 of 2560): 29 us each, cut 14 and 16; a step of that layer
// 419 us against 268, of 512 tokens of h 3072 437 against 411, with both gradients of a layer as launches of their own.
template <bool AK, bool BK_, bool FAR, TileForm FORM>
__global__ void __launch_bounds__((tile_threads<kT64>), (tile_waves_per_simd<kT64>)) gemm_serial_kernel(MfmaGemmArgs g) {
  using T = TileShape<kT64, AK && BK_>;
  gemm_tile<AK, BK_, T::BM, T::BN, FORM, false, T::S, true, T::BK, T::waves, true, FAR>(g, blockIdx.x, 0);
}

template <bool AK, bool BK_, bool FAR = false, TileForm FORM = kSingle>
hipError_t launch_serial(bool far, MfmaGemmArgs a, hipStream_t st) {
  if (far && !FAR) return launch_serial<AK, BK_, true>(far, a, st);
  if constexpr (AK && BK_ && FORM == kSingle)
    if (a.epi == kEpiGelu) return launch_serial<AK, BK_, FAR, kWithGelu>(far, a, st);
  using T = TileShape<kT64, AK && BK_>;
  static_assert(kMaxBK % T::BK == 0, "ranges are whole slabs");
  constexpr size_t smem = tile_lds<T>;
  auto kern = gemm_serial_kernel<AK, BK_, FAR, FORM>;
  LYNX_RAISE_LDS_LIMIT(kern, smem);
  set_tiles(&a, T::BM, T::BN);
  hipLaunchKernelGGL(kern, dim3(a.tiles_m * a.tiles_n), dim3(T::waves * kWave), smem, st, a);
  return hipGetLastError();
}

// The two products over a seq x seq gradient, dQ = dS K and dK = dS^T Q, in one launch: a workgroup of each in turn,
// longest contractions first.  `by_slice`: slice z on XCD z % 8, one slice after the other, so that whichever of
// the two comes second finds that slice of dS in the caches; otherwise all slices' longest tiles first.
template <int TILE, bool FAR>
__global__ void __launch_bounds__((tile_threads<TILE>), (tile_waves_per_simd<TILE>))
attn_gradients_kernel(MfmaGemmArgs rows, MfmaGemmArgs cols, int by_slice) {
  using T = TileShape<TILE, false>;
  const int x = static_cast<int>(blockIdx.x), per_slice = 2 * rows.tiles_m * rows.tiles_n;
  int z, w;
  if (by_slice) {
    const int y = x >> 3;
    z = y / per_slice * 8 + (x & 7);
    w = y % per_slice;
    if (z >= rows.nz) return;
  } else {
    w = x / rows.nz;
    z = x - w * rows.nz;
  }
  const int tile = (w >> 1) * rows.nz + z;
  if (w & 1) gemm_tile<false, false, T::BM, T::BN, kOfSequence, false, T::S, true, T::BK, T::waves, false, FAR>(cols, tile, 0);
  else gemm_tile<true, false, T::BM, T::BN, kOfSequence, false, T::S, true, T::BK, T::waves, false, FAR>(rows, tile, 0);
}

template <int TILE, bool FAR = false>
hipError_t launch_attn_gradients(MfmaGemmArgs rows, MfmaGemmArgs cols, hipStream_t st) {
  using T = TileShape<TILE, false>;
  constexpr size_t smem = tile_lds<T>;
  auto kern = attn_gradients_kernel<TILE, FAR>;
  LYNX_RAISE_LDS_LIMIT(kern, smem);
  for (MfmaGemmArgs* g : {&rows, &cols}) {
    set_tiles(g, T::BM, T::BN);
  }
  const int per_slice = 2 * rows.tiles_m * rows.tiles_n;
  // From eight slices per XCD on, the idle end of the last one is a small part.  Slice by slice and all at once: 64
  // slices of s = 2048 142 and 161 us, 128 of 1024 59 and 63; but 40 of 2048 87 and 84, 32 of 2048 79 and 68.
  // (Two launches: 182, 66, 97 and 89.)
  const bool by_slice = rows.nz >= 64;
  const int groups = by_slice ? 8 * ceil_div(rows.nz, 8) * per_slice : rows.nz * per_slice;
  hipLaunchKernelGGL(kern, dim3(groups), dim3(T::waves * kWave), smem, st, rows, cols, by_slice ? 1 : 0);
  return hipGetLastError();
}

template <int TILE, bool FAR = false>
hipError_t launch_ragged_pair(MfmaGemmArgs w, MfmaGemmArgs d, const ColumnSumInput* in, hipStream_t st) {
  using T = TileShape<TILE, false>;
  constexpr size_t smem = tile_lds<T>;
  for (MfmaGemmArgs* g : {&w, &d}) set_tiles(g, T::BM, T::BN);
  const int n_w = w.tiles_m * w.tiles_n * w.k_splits, n_d = d.tiles_m * d.tiles_n * d.k_splits;
  const int dgrad_first = d.k_per > w.k_per;
  const int n_first = dgrad_first ? n_d : n_w, n_pad = (n_first + 7) & ~7;
  const int n = n_pad + n_w + n_d - n_first;
  if constexpr (TILE == kT64) {
    if (in != nullptr) {
      auto kern = gemm_ragged_pair_guest_kernel<TILE, FAR>;
      LYNX_RAISE_LDS_LIMIT(kern, smem);
      const ColumnPartials guest = guest_partials(*in, n_pad, n, T::waves);
      hipLaunchKernelGGL(kern, dim3(n + guest.end - guest.first), dim3(T::waves * kWave), smem, st, w, d, n_first, dgrad_first, guest);
      return hipGetLastError();
    }
  }
  auto kern = gemm_ragged_pair_kernel<TILE, FAR>;
  LYNX_RAISE_LDS_LIMIT(kern, smem);
  hipLaunchKernelGGL(kern, dim3(n), dim3(T::waves * kWave), smem, st, w, d, n_first, dgrad_first);
  return hipGetLastError();
}

// C = round(sum over the K ranges, in range order, of partial[range][m][n] (+ bias)), and what the
// product's epilogue does with it (GemmEpilogueKind: none, GeLU, or bias + dropout + residual), for one or
// two products: the first `n0` workgroups belong to `a`, the rest to `b`.
__global__ void __launch_bounds__(256) splitk_finish_kernel(MfmaGemmArgs a, MfmaGemmArgs b, int n0) {
  const bool second = static_cast<int>(blockIdx.x) >= n0;
  const MfmaGemmArgs& g = second ? b : a;
  const long long v = static_cast<long long>(blockIdx.x - (second ? n0 : 0)) * 256 + threadIdx.x;  // 8 consecutive n
  const int per_row = g.N / 8;
  if (v >= static_cast<long long>(g.M) * per_row) return;
  const int m = static_cast<int>(v / per_row), n = static_cast<int>(v - static_cast<long long>(m) * per_row) * 8;
  const float* p = g.partial + static_cast<long long>(m) * g.N + n;
  float s[8];
  load8(p, s);
  for (int sp = 1; sp < g.k_splits; ++sp) {
    p += static_cast<long long>(g.M) * g.N;
    float t[8];
    load8(p, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] += t[i];
  }
  if (g.bias != nullptr) {
    float t[8];
    load8(g.bias + n, t);
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] += t[i];
  }
  bf16_t* c = g.C + static_cast<long long>(m) * g.ldc + n;
  if (g.epi == kEpiNone) {
    store8(c, s);
    return;
  }
  float vec[8], x[8], o[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) s[i] = round_to_storage(s[i], static_cast<bf16_t*>(nullptr));
  if (g.plain != nullptr) store8(g.plain + static_cast<long long>(m) * g.ldc + n, s);
  if (g.epi == kEpiGelu) {
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = gelu_f(s[i]);
    store8(c, o);
    return;
  }
  load8(g.vec + n, vec);
  load8(g.aux + static_cast<long long>(m) * g.aux_ld + n, x);
  bias_dropout_add8(s, vec, x, g.key, (static_cast<uint64_t>(m) * static_cast<uint64_t>(g.N) + n) >> 3, o);
  store8(c, o);
}

hipError_t launch_finish(const MfmaGemmArgs* a, const MfmaGemmArgs* b, hipStream_t st) {
  auto groups = [](const MfmaGemmArgs* g) { return static_cast<int>((static_cast<long long>(g->M) * (g->N / 8) + 255) / 256); };
  const int n0 = groups(a), n1 = b != nullptr ? groups(b) : 0;
  hipLaunchKernelGGL(splitk_finish_kernel, dim3(n0 + n1), dim3(256), 0, st, *a, b != nullptr ? *b : *a, n0);
  return hipGetLastError();
}

struct RaggedPairPlan {
  int tile, w_per, d_per;   // indices per K range of the weight gradient, of the input gradient
  double us;
};

size_t partial_bytes(int M, int N, int splits) {
  return splits > 1 ? static_cast<size_t>(splits) * M * N * sizeof(float) : 0;
}

// us of a pair launch: the units share the work of both products; a unit cannot be done before its
// longest workgroup is, which has a neighbour for part of its time, and on average half of a short
// workgroup is left over at the end.
double pair_cost(const TileCost& t, const GemmDesc& w, int w_per, const GemmDesc& d, int d_per) {
  const int ws = ceil_div(w.K, w_per), ds = ceil_div(d.K, d_per);
  const double nw = static_cast<double>(ceil_div(w.M, t.bm)) * ceil_div(w.N, t.bn) * ws;
  const double nd = static_cast<double>(ceil_div(d.M, t.bm)) * ceil_div(d.N, t.bn) * ds;
  const double sw = ceil_div(w_per < w.K ? w_per : w.K, 32), sd = ceil_div(d_per < d.K ? d_per : d.K, 32);
  const double n = nw + nd, round = static_cast<double>(TileCost::kUnits) * t.share;
  const double rate = t.slab(n < round ? n : round);            // of a round as full as this launch's
  const double at_once = n < round ? n : round;
  const double even = (nw * sw + nd * sd) * rate / at_once + (n > round ? 0.42 * (sw < sd ? sw : sd) * rate : 0.0);
  const double longest = (sw > sd ? sw : sd) * (n <= round ? rate : 0.86 * t.one_each + 0.14 * t.full);
  double us = t.fixed * (1.0 + 0.48 * n / round) + (longest > even ? longest : even);
  const double bytes = static_cast<double>(partial_bytes(w.M, w.N, ws) + partial_bytes(d.M, d.N, ds));
  if (bytes > 0.0) us += kFinishFixed[1] + bytes / kFinishBytesPerUs[1];
  return us;
}

RaggedPairPlan search_pair(const GemmDesc& w, const GemmDesc& d) {
  // (the GeLU epilogue's column sums are formed tile by tile, so such an input gradient is not cut)
  const bool cut_d = d.epi.kind == kEpiNone;
  RaggedPairPlan best{kT64, range_of(w.K, 1), range_of(d.K, 1), 1e30};
  const bool far = w.M >= kFarStride || w.N >= kFarStride || d.N >= kFarStride || d.K >= kFarStride;  // the row strides
  // Partial sums take at most three times what the tokens' side of both products does, or 8 MB: more of them named
  // workspaces up to 1.7 times as large, and is not faster (582 pairs as above: 2.0 % over the fastest either way).
  const size_t tokens_bytes = 2 * static_cast<size_t>(d.M) * (static_cast<size_t>(d.N) + d.K);
  const size_t most_bytes = 3 * tokens_bytes > (8u << 20) ? 3 * tokens_bytes : (8u << 20);
  int per[2][sizeof(kCuts) / sizeof(kCuts[0])], n[2] = {0, 0};  // the distinct ranges of the two contractions
  for (int which = 0; which < 2; ++which)
    for (int cut : kCuts) {
      const int K = which == 0 ? w.K : d.K;
      if (cut > 1 && (K < kMinRange * cut || (which == 1 && !cut_d))) break;
      const int range = range_of(K, cut);
      if (n[which] == 0 || range != per[which][n[which] - 1]) per[which][n[which]++] = range;
    }
  for (int iw = 0; iw < n[0]; ++iw)
    for (int id = 0; id < n[1]; ++id) {
      const int ws = ceil_div(w.K, per[0][iw]), ds = ceil_div(d.K, per[1][id]);
      if (partial_bytes(w.M, w.N, ws) + partial_bytes(d.M, d.N, ds) > most_bytes) continue;
      for (int t = far ? kT64 : 0; t < kNumRaggedTiles; ++t) {
        if (t == kT128x64) continue;   // (no pair kernel of this tile)
        const double us = pair_cost(kPairCost[t], w, per[0][iw], d, per[1][id]);
        if (us < best.us) best = {t, per[0][iw], per[1][id], us};
      }
    }
  return best;
}

RaggedPairPlan plan_pair_ragged(const GemmDesc& w, const GemmDesc& d) {
  static thread_local PlanCache<RaggedPairPlan, 7> cache;
  return cache.get({w.M, w.N, w.K, d.M, d.N, d.K, d.epi.kind}, [&] { return search_pair(w, d); });
}

}  // namespace

RaggedChoice ragged_product(const GemmDesc& d) {
  const ProductPlan p = plan_product(d);
  const int splits = p.splits(d.K);
  return {p.us, partial_bytes(d.M, d.N, splits), 0, kProductCost[p.tile].bm, kProductCost[p.tile].bn, splits, 1};
}

int attention_tile(const GemmDesc& d, long long workgroups_per_tile) {
  const int tile = d.causal == kCausalOutLower || d.N > 64 ? kT128 : kT128x64;
  const TileCost& t = kProductCost[tile];
  return ceil_div(d.M, t.bm) * ceil_div(d.N, t.bn) * workgroups_per_tile < TileCost::kUnits ? kT64 : tile;
}

bool gemm_attention_pair_joint(const GemmDesc& rows) {
  const long long slices = static_cast<long long>(rows.nz1) * rows.nz2;
  const TileCost& t = kProductCost[is_far(rows) ? kT64 : attention_tile(rows, slices)];
  return fits_grid((slices + 7) / 8 * 16 * ceil_div(rows.M, t.bm) * ceil_div(rows.N, t.bn), 4 * kWave);
}

hipError_t gemm_attention_pair(const GemmDesc& rows, const GemmDesc& cols, hipStream_t st) {
  const MfmaGemmArgs r = make_args(rows), c = make_args(cols);
  if (!gemm_attention_pair_joint(rows)) {
    const hipError_t e = gemm_attention(rows, st);
    return e != hipSuccess ? e : gemm_attention(cols, st);
  }
  if (is_far(rows) || is_far(cols)) return launch_attn_gradients<kT64, true>(r, c, st);
  switch (attention_tile(rows, r.nz)) {
    case kT128: return launch_attn_gradients<kT128>(r, c, st);
    case kT128x64: return launch_attn_gradients<kT128x64>(r, c, st);
    default: return launch_attn_gradients<kT64>(r, c, st);
  }
}

hipError_t gemm_ragged(const GemmDesc& d, float* scratch, size_t scratch_bytes, hipStream_t st) {
  MfmaGemmArgs a = make_args(d);
  const bool a_k = d.a_sk == 1, b_k = d.b_sk == 1, far = is_far(d);
  int tile;
  if (d.causal == kCausalNone && a.nz == 1) {
    const ProductPlan p = plan_product(d);
    tile = p.tile;
    if (p.splits(d.K) > 1 && d.serial) {
      a.k_per = p.k_per;
      if (!a_k || !b_k) return hipErrorInvalidValue;  // (gradients come in pairs)
      return launch_serial<true, true>(far, a, st);
    }
    if (p.splits(d.K) > 1) {
      // the cut is part of the shape's summation order: no silent change where scratch is short
      if (scratch == nullptr || scratch_bytes < partial_bytes(d.M, d.N, p.splits(d.K))) return hipErrorInvalidValue;
      a.k_splits = p.splits(d.K);
      a.k_per = p.k_per;
      a.partial = scratch;
    }
  } else {
    // attention products: up to 128 rows (the zero padding of the seq x seq operands reaches the next
    // multiple of 128), a head dimension of up to 64 is half a tile wide, and where that leaves compute
    // units without a workgroup, 64 x 64 (21 slices of s = 328, d = 104: 10.2 us with 128 x 128 tiles)
    tile = attention_tile(d, a.nz);
  }
  hipError_t e;
  if (a_k && b_k) e = launch_tile<true, true>(tile, far, a, st);
  else if (a_k) e = launch_tile<true, false>(tile, far, a, st);
  else if (!b_k) e = launch_tile<false, false>(tile, far, a, st);
  else return hipErrorInvalidValue;
  if (e != hipSuccess || a.k_splits == 1) return e;
  return launch_finish(&a, nullptr, st);
}

RaggedChoice ragged_pair(const GemmDesc& dgrad, const GemmDesc& wgrad) {
  const RaggedPairPlan p = plan_pair_ragged(wgrad, dgrad);
  const int ws = ceil_div(wgrad.K, p.w_per), ds = ceil_div(dgrad.K, p.d_per);
  return {p.us, partial_bytes(wgrad.M, wgrad.N, ws) + partial_bytes(dgrad.M, dgrad.N, ds),
          ceil_div(dgrad.M, kTileWaveRows[p.tile]), kPairCost[p.tile].bm, kPairCost[p.tile].bn, ws, ds};
}

hipError_t gemm_ragged_pair(const GemmDesc& dgrad, const GemmDesc& wgrad, float* scratch, size_t scratch_bytes,
                            const ColumnSumInput* in, ColumnSums* sums, hipStream_t st) {
  const RaggedPairPlan p = plan_pair_ragged(wgrad, dgrad);
  MfmaGemmArgs d = make_args(dgrad), w = make_args(wgrad);
  w.k_splits = ceil_div(w.K, p.w_per);
  w.k_per = p.w_per;
  d.k_splits = ceil_div(d.K, p.d_per);
  d.k_per = p.d_per;
  const size_t w_bytes = partial_bytes(w.M, w.N, w.k_splits), d_bytes = partial_bytes(d.M, d.N, d.k_splits);
  const int colsum_rows = ceil_div(dgrad.M, kTileWaveRows[p.tile]);
  // columns whose GeLU partials have room at once
  int at_once = dgrad.N;
  if (dgrad.epi.kind == kEpiGeluBwd) {
    const size_t room = dgrad.epi.colsum_bytes / (static_cast<size_t>(colsum_rows) * sizeof(float));
    if (room < static_cast<size_t>(dgrad.N)) at_once = static_cast<int>(room) / 8 * 8;
    if (at_once == 0) return hipErrorInvalidValue;
    if (at_once < dgrad.N && at_once > 256) at_once = at_once / 256 * 256;  // whole tiles
  }
  const bool in_parts = at_once < dgrad.N, far = is_far(dgrad) || is_far(wgrad);
  const bool serial = dgrad.serial && w_bytes + d_bytes > 0;
  if (in_parts && !dgrad.serial && w_bytes > 0) return hipErrorInvalidValue;
  if (in != nullptr && (serial || in_parts || p.tile != kT64)) return hipErrorInvalidValue;
  if (w_bytes + d_bytes > 0 && !serial && (scratch == nullptr || scratch_bytes < w_bytes + d_bytes)) return hipErrorInvalidValue;
  hipError_t e;
  if (serial || in_parts) {
    // (the product that is not cut in the plan's tile: the GeLU epilogue's column partials depend on it)
    const bool w_cut = w.k_splits > 1, d_cut = d.k_splits > 1;
    w.k_splits = d.k_splits = 1;
    const int w_tile = p.tile == kT256 || p.tile == kT256x128 ? kT128 : p.tile;  // (no larger one for two MN-major operands)
    e = w_cut ? launch_serial<false, false>(far, w, st) : launch_tile<false, false>(w_tile, far, w, st);
    if (in_parts) {
      for (int n0 = 0; e == hipSuccess && n0 < dgrad.N; n0 += at_once) {
        MfmaGemmArgs part = d;
        part.N = n0 + at_once < dgrad.N ? at_once : dgrad.N - n0;
        part.B = d.B + n0;
        part.C = d.C + n0;
        part.aux = d.aux + n0;
        e = launch_tile<true, false>(p.tile, far, part, st);
        ColumnSums of_part;
        if (e == hipSuccess) e = of_part.add(part.colsum_partial, static_cast<bf16_t*>(dgrad.epi.colsum_out) + n0, colsum_rows, part.N);
        if (e == hipSuccess) e = finish_column_sums(1, &of_part, st);
      }
      return e;
    }
    if (e == hipSuccess) e = d_cut ? launch_serial<true, false>(far, d, st) : launch_tile<true, false>(p.tile, far, d, st);
  } else {
    w.partial = scratch;
    d.partial = scratch + w_bytes / sizeof(float);
    switch (p.tile) {
      case kT256: e = launch_ragged_pair<kT256>(w, d, nullptr, st); break;
      case kT256x128: e = launch_ragged_pair<kT256x128>(w, d, nullptr, st); break;
      case kT128: e = launch_ragged_pair<kT128>(w, d, nullptr, st); break;
      default: e = far ? launch_ragged_pair<kT64, true>(w, d, in, st) : launch_ragged_pair<kT64>(w, d, in, st); break;
    }
    if (e == hipSuccess && in != nullptr) e = sums->add(in->part, in->out, (in->rows + kPartialRows - 1) / kPartialRows, in->cols);
  }
  if (e != hipSuccess) return e;
  if (w.k_splits > 1 && d.k_splits > 1) e = launch_finish(&w, &d, st);
  else if (w.k_splits > 1) e = launch_finish(&w, nullptr, st);
  else if (d.k_splits > 1) e = launch_finish(&d, nullptr, st);
  if (e != hipSuccess || dgrad.epi.kind != kEpiGeluBwd) return e;
  return sums->add(dgrad.epi.colsum_partial, dgrad.epi.colsum_out, colsum_rows, dgrad.N);
}

}  // namespace lynx
