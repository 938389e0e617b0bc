// bf16 matrix products of attention: kernels and launches (the tile of those that contract over tokens is
// gemm_tile.h; linear products: gemm_ragged.hip).
#include <mutex>

#include "gemm_launch.h"

namespace lynx {
namespace {

// The products of attention with the seq x seq operand: memory-bound.  128 x 128 tiles: the zero
// padding of that operand reaches the next multiple of 128 only, and two workgroups fit a compute
// unit (one loads while the other stores).
template <bool A_KMAJOR>
__global__ void __launch_bounds__(kThreads, 2) attn_product_kernel(MfmaGemmArgs g) {
  gemm_tile<A_KMAJOR, false, 128, 128, kOfSequence>(g, blockIdx.x, 0);
}

// Work items of the score-shaped row-block kernels: row block tm (128 rows) owns tiles
// tn = 0..tm; it is cut into runs of at most `run` tiles, one workgroup each, so that no
// workgroup walks more than `run` tiles (a workgroup per whole row block leaves the launch
// waiting for the 16-tile blocks while most compute units have run out of work).  Items are
// numbered longest row block first; item * nz + z is the workgroup of matrix z.
//
// Runs of four tiles share the A tile and hide the loads of the next B tile; where they would
// not give every compute unit its two workgroups, a short launch is what counts: runs of two or one
// (8 slices of s = 384, dS: 24 workgroups of up to three tiles 17.3 us, 48 of one 10.5).
constexpr int kAttnRun = 4;
__host__ __device__ inline int attn_runs_of(int tm, int run) { return (tm + run) / run; }
inline int attn_items(int tiles_m, int run) {
  int n = 0;
  for (int tm = 0; tm < tiles_m; ++tm) n += attn_runs_of(tm, run);
  return n;
}
inline int attn_run(int tiles_m, int nz) {
  int run = kAttnRun;
  while (run > 1 && static_cast<long long>(attn_items(tiles_m, run)) * nz < 512) run /= 2;
  return run;
}
// item -> (tm, first tile, one past the last tile)
__device__ __forceinline__ void attn_item(int item, int tiles_m, int run, int& tm, int& tn0, int& tn1) {
  tm = tiles_m - 1;
  while (tm > 0 && item >= attn_runs_of(tm, run)) {
    item -= attn_runs_of(tm, run);
    --tm;
  }
  tn0 = item * run;
  tn1 = min(tn0 + run, tm + 1);
}

// Score-shaped batched products with a short contraction (S = Q K^T, dPd = dC V^T: K = head
// dimension), lower triangle only.  A tile of such a product is all latency: load two small
// operand tiles, 32 MFMAs per wavefront, store 32 KB.  Here a workgroup owns a run of tiles of
// one block of 128 rows of one matrix: the A tile stays in LDS; the one B buffer doubles as
// the staging area of the store pass, the next B tile is requested as soon as every wavefront
// has its rows back in registers, and the stores are never waited for.  At 64 KB of LDS (head
// dimension 128) two workgroups share a compute unit: one loads and stores while the other
// multiplies.
//
// RAGGED: the sequence is not a multiple of 128 or the head dimension not KD.  Row i >= s repeats row
// s - 1 of A and row s - 8 + i % 8 of B, and what they produce is stored where the original went:
// the same values twice, so no access needs a mask and the waits can be counted.  Chunks of the
// contraction beyond the head dimension read zeros.
__device__ __forceinline__ int repeat_row(int i, int s) { return min(i, s - 1); }
__device__ __forceinline__ int repeat_octet(int i, int s) { return min(i, s - 8 + (i & 7)); }

// One 128 x KD operand tile whose first row is row0 of the matrix at `base`, row stride ld.
template <int KD, bool RAGGED, bool OCTET>
__device__ __forceinline__ void load_score_tile(const bf16_t* base, long long ld, int row0, int rows, int head_dim,
                                                bf16_t* dst, int wave, int lane) {
  using SL = Slab<128, true>;
#pragma unroll
  for (int sl = 0; sl < KD / kBK; ++sl)
#pragma unroll
    for (int j = 0; j < SL::kLoadsPerWave; ++j) {
      int row = row0 + SL::lane_mn(wave, j, lane);
      const int k = sl * kBK + SL::lane_k(wave, j, lane);
      if (RAGGED) row = OCTET ? repeat_octet(row, rows) : repeat_row(row, rows);
      const bf16_t* from = base + row * ld + k;
      if (RAGGED && k >= head_dim) from = reinterpret_cast<const bf16_t*>(&kZeroChunk);
      __builtin_amdgcn_global_load_lds((global_void_ptr)(from),
                                       (lds_void_ptr)(dst + sl * SL::kElems + SL::lds_offset(wave, j)), 16, 0, 0);
    }
}

template <int KD, bool RAGGED>
__global__ void __launch_bounds__(kThreads, 2) attn_outer_kernel(MfmaGemmArgs g) {
  constexpr int WM = 64, WN = 64, TM = 2, TN = 2;
  constexpr int kSlabs = KD / kBK;
  using SL = Slab<128, true>;
  constexpr int kOpElems = kSlabs * SL::kElems;       // one 128 x KD operand tile
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* sA = reinterpret_cast<bf16_t*>(smem_raw);
  bf16_t* sB = sA + kOpElems;                           // B tile, then 4 x (64 x 64) of staging

  const int item = blockIdx.x / g.nz;
  const int bz = blockIdx.x - item * g.nz;
  int tm, tn0, tn1;
  attn_item(item, g.tiles_m, g.run, tm, tn0, tn1);
  const int z1 = bz / g.nz2, z2 = bz - z1 * g.nz2;
  const bf16_t* Abase = g.A + z1 * g.a_z1 + z2 * g.a_z2;
  const bf16_t* Bbase = g.B + z1 * g.b_z1 + z2 * g.b_z2;
  bf16_t* Cbase = g.C + z1 * g.c_z1 + z2 * g.c_z2;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * WN;

  load_score_tile<KD, RAGGED, false>(Abase, g.lda, tm * 128, g.M, g.K, sA, wave, lane);
  load_score_tile<KD, RAGGED, true>(Bbase, g.ldb, tn0 * 128, g.M, g.K, sB, wave, lane);

  constexpr int kRowChunks = WN / 8;                    // 8
  constexpr int kRowsPerStore = kWave / kRowChunks;     // 8
  constexpr int kStores = WM / kRowsPerStore;           // 8 stores per wavefront per tile
  bf16_t* stage = sB + wave * (WM * WN);
  const int lr = lane / kRowChunks, lc = lane % kRowChunks;

  // S is read once, by the softmax: streaming stores, unless a row's end shares its 128-byte line with the
  // next row's beginning (s = 1000, 100 slices: 68 us with the hint, 35 without)
  const bool streaming = !RAGGED || g.ldc % 64 == 0;
  for (int tn = tn0; tn < tn1; ++tn) {
    // B(tn) (and, the first time, A) has landed: everything older than the previous tile's stores
    if (tn == tn0) wait_vmcnt<0>();
    else wait_vmcnt<kStores>();
    block_barrier();

    floatx16_t acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KD / 16; ++kk) {
      Frag<true> fa[TM], fb[TN];
#pragma unroll
      for (int j = 0; j < TM; ++j) fa[j] = SL::fragment(sA + (kk >> 1) * SL::kElems, wm0 + 32 * j, kk & 1, lane);
#pragma unroll
      for (int i = 0; i < TN; ++i) fb[i] = SL::fragment(sB + (kk >> 1) * SL::kElems, wn0 + 32 * i, kk & 1, lane);
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[i].operand(), fa[j].operand(), acc[i][j], 0, 0, 0);
    }
    block_barrier();  // every wavefront has read B(tn): its buffer becomes the staging area
    // round into this wavefront's staging region, then whole rows back, 16 bytes per lane
    // (acc[i][j][r]: n = wn0 + 32 i + 8 (r / 4) + 4 (lane / 32) + r % 4, m = wm0 + 32 j + lane % 32)
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nl = 32 * i + 8 * q + 4 * (lane >> 5);
#pragma unroll
        for (int j = 0; j < TM; ++j) {
          const int ml = 32 * j + (lane & 31);
          uintx2_t o;
          o[0] = pack_bf16(acc[i][j][4 * q + 0], acc[i][j][4 * q + 1]);
          o[1] = pack_bf16(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
          const int chunk = (nl >> 3) ^ (ml & (kRowChunks - 1));
          // As inline assembly: a store to LDS that the compiler sees is made to wait for
          // every direct-to-LDS load in flight and, with them, for the previous tile's
          // stores.  LDS executes a wavefront's accesses in order, so the row reads below
          // see these writes.
          typedef __attribute__((address_space(3))) bf16_t* lds_ptr_t;
          const uint32_t addr = static_cast<uint32_t>(
              reinterpret_cast<uintptr_t>((lds_ptr_t)(stage + ml * WN + chunk * 8 + (nl & 7))));
          asm volatile("ds_write_b64 %0, %1" : : "v"(addr), "v"(o) : "memory");
        }
      }
    uintx4_t rows[kStores];
#pragma unroll
    for (int u = 0; u < kStores; ++u) {
      const int r = u * kRowsPerStore + lr;
      typedef const __attribute__((address_space(3))) bf16_t* lds_cptr_t;
      const uint32_t addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
          (lds_cptr_t)(stage + r * WN + ((lc ^ (r & (kRowChunks - 1))) << 3))));
      asm volatile("ds_read_b128 %0, %1" : "=v"(rows[u]) : "v"(addr) : "memory");
    }
    wait_lgkmcnt0();
#pragma unroll
    for (int u = 0; u < kStores; ++u) asm volatile("" : "+v"(rows[u]));
    block_barrier();  // every wavefront has its rows: the buffer can take the next B tile
    if (tn + 1 < tn1) load_score_tile<KD, RAGGED, true>(Bbase, g.ldb, (tn + 1) * 128, g.M, g.K, sB, wave, lane);
    int col = tn * 128 + wn0 + lc * 8;
    if (RAGGED) col = repeat_octet(col, g.M);
#pragma unroll
    for (int u = 0; u < kStores; ++u) {
      int r = tm * 128 + wm0 + u * kRowsPerStore + lr;
      if (RAGGED) r = repeat_row(r, g.M);
      uintx4_t* dst = reinterpret_cast<uintx4_t*>(Cbase + static_cast<long long>(r) * g.ldc + col);
      if (streaming) __builtin_nontemporal_store(rows[u], dst);
      else *dst = rows[u];
    }
  }
}

// dS from dC, V and P in one launch: the score-shaped product dPd = dC V^T with the backward
// of dropout and softmax (B5 + B4) in its store pass, so dPd is never written:
//   dS = scale P (keep c round(dPd) - dot),  dot_i = sum_j dP_ij P_ij.
// The row dot product comes in from a small kernel that forms it as sum_dd dC[i, dd] C[i, dd]
// (= sum_j dPd_ij Pd_ij since Pd V = C: the same number up to the rounding of Pd and dPd), so
// one pass over the tiles suffices.  Same walk as attn_outer_kernel (a workgroup owns a block
// of 128 rows, the A tile stays in LDS), but the store pass is long here (a Philox call per
// 8 elements), so: one B buffer, which doubles as the staging area; the next B tile and the
// next tile's vectors of P are requested just before the store pass and arrive during it;
// and the 64 KB of LDS let two workgroups share a compute unit.  The loads of P are inline
// assembly with waits counted by hand: loads the compiler tracks would be waited for at
// the loop's back edge together with everything issued after them.
__global__ void __launch_bounds__(kThreads, 2) attn_dscores_kernel(MfmaGemmArgs g) {
  constexpr int KD = 128;
  constexpr int WM = 64, WN = 64, TM = 2, TN = 2;
  constexpr int kSlabs = KD / kBK;
  using SL = Slab<128, true>;
  constexpr int kOpElems = kSlabs * SL::kElems;  // one 128 x KD operand tile
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* sA = reinterpret_cast<bf16_t*>(smem_raw);
  bf16_t* sB = sA + kOpElems;

  const int item = blockIdx.x / g.nz;
  const int bz = blockIdx.x - item * g.nz;
  int tm, tn0, tn1;
  attn_item(item, g.tiles_m, g.run, tm, tn0, tn1);
  const int z1 = bz / g.nz2, z2 = bz - z1 * g.nz2;
  const bf16_t* Abase = g.A + z1 * g.a_z1 + z2 * g.a_z2;
  const bf16_t* Bbase = g.B + z1 * g.b_z1 + z2 * g.b_z2;
  bf16_t* Cbase = g.C + z1 * g.c_z1 + z2 * g.c_z2;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave >> 1) * WM, wn0 = (wave & 1) * WN;

  constexpr int kTileLoads = kSlabs * SL::kLoadsPerWave;  // direct loads per wavefront per tile
  load_score_tile<KD, false, false>(Abase, g.lda, tm * 128, g.M, g.K, sA, wave, lane);
  load_score_tile<KD, false, true>(Bbase, g.ldb, tn0 * 128, g.M, g.K, sB, wave, lane);

  constexpr int kRowChunks = WN / 8;                 // 8
  constexpr int kRowsPerStore = kWave / kRowChunks;  // 8
  constexpr int kStores = WM / kRowsPerStore;        // 8 rows of P / stores per lane per tile
  bf16_t* stage = sB + wave * (WM * WN);
  const int lr = lane / kRowChunks, lc = lane % kRowChunks;

  // this lane's eight rows: dot products, dropout indices, vectors of P (two sets)
  const bf16_t* Pbase = g.aux + z1 * g.c_z1 + z2 * g.c_z2;
  auto row_of = [&](int u) { return tm * 128 + wm0 + u * kRowsPerStore + lr; };
  auto col_of = [&](int tn) { return tn * 128 + wn0 + lc * 8; };
  const uint64_t rows_before = (static_cast<uint64_t>(z1) * g.global_heads + g.head0 + z2) * g.M;
  float dot[kStores];
  uint64_t gidx[kStores];
  uintx4_t p0[kStores], p1[kStores];
  auto request_p = [&](int tn, uintx4_t (&pv)[kStores]) {
#pragma unroll
    for (int u = 0; u < kStores; ++u) {
      const bf16_t* src = Pbase + static_cast<long long>(row_of(u)) * g.ldc + col_of(tn);
      asm volatile("global_load_dwordx4 %0, %1, off nt" : "=v"(pv[u]) : "v"(src) : "memory");
    }
  };
  request_p(tn0, p0);
#pragma unroll
  for (int u = 0; u < kStores; ++u) {
    const int i = row_of(u);
    dot[u] = g.rowdot[static_cast<long long>(bz) * g.M + i];
    gidx[u] = (rows_before + i) * static_cast<uint64_t>(g.N);
  }
  // (a use: the compiler waits for these loads here, once, and tracks nothing into the loop)
#pragma unroll
  for (int u = 0; u < kStores; ++u) asm volatile("" : "+v"(dot[u]));

  // One tile; `pc` holds this tile's vectors of P, `pn` receives the next tile's.
  auto tile_step = [&](const int tn, uintx4_t (&pc)[kStores], uintx4_t (&pn)[kStores]) {
    // B(tn) has landed.  Issued after it: the previous step's requests for P and its stores
    // (nothing the first time, when everything issued so far is waited for).
    if (tn == tn0) wait_vmcnt<0>();
    else wait_vmcnt<2 * kStores>();
    block_barrier();
    floatx16_t acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KD / 16; ++kk) {
      Frag<true> fa[TM], fb[TN];
#pragma unroll
      for (int j = 0; j < TM; ++j) fa[j] = SL::fragment(sA + (kk >> 1) * SL::kElems, wm0 + 32 * j, kk & 1, lane);
#pragma unroll
      for (int i = 0; i < TN; ++i) fb[i] = SL::fragment(sB + (kk >> 1) * SL::kElems, wn0 + 32 * i, kk & 1, lane);
#pragma unroll
      for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[i].operand(), fa[j].operand(), acc[i][j], 0, 0, 0);
    }
    block_barrier();  // every wavefront has read B(tn): its buffer becomes the staging area
    // round into this wavefront's quarter, read whole rows back, 16 bytes per lane
    // (acc[i][j][r]: n = wn0 + 32 i + 8 (r / 4) + 4 (lane / 32) + r % 4, m = wm0 + 32 j + lane % 32)
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nl = 32 * i + 8 * q + 4 * (lane >> 5);
#pragma unroll
        for (int j = 0; j < TM; ++j) {
          const int ml = 32 * j + (lane & 31);
          uintx2_t o;
          o[0] = pack_bf16(acc[i][j][4 * q + 0], acc[i][j][4 * q + 1]);
          o[1] = pack_bf16(acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
          const int chunk = (nl >> 3) ^ (ml & (kRowChunks - 1));
          typedef __attribute__((address_space(3))) bf16_t* lds_ptr_t;
          const uint32_t addr = static_cast<uint32_t>(
              reinterpret_cast<uintptr_t>((lds_ptr_t)(stage + ml * WN + chunk * 8 + (nl & 7))));
          asm volatile("ds_write_b64 %0, %1" : : "v"(addr), "v"(o) : "memory");
        }
      }
    uintx4_t rows[kStores];
#pragma unroll
    for (int u = 0; u < kStores; ++u) {
      const int r = u * kRowsPerStore + lr;
      typedef const __attribute__((address_space(3))) bf16_t* lds_cptr_t;
      const uint32_t addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(
          (lds_cptr_t)(stage + r * WN + ((lc ^ (r & (kRowChunks - 1))) << 3))));
      asm volatile("ds_read_b128 %0, %1" : "=v"(rows[u]) : "v"(addr) : "memory");
    }
    wait_lgkmcnt0();
#pragma unroll
    for (int u = 0; u < kStores; ++u) asm volatile("" : "+v"(rows[u]));
    block_barrier();  // every wavefront has its rows: the buffer can take the next B tile
    if (tn + 1 < tn1) {
      load_score_tile<KD, false, true>(Bbase, g.ldb, (tn + 1) * 128, g.M, g.K, sB, wave, lane);
      request_p(tn + 1, pn);
    }
    // this tile's P: requested a step ago; issued since: the previous step's stores and, if
    // there is a next tile, its B tile and its P
    if (tn == tn0) {
      // (waited for at the top)
    } else if (tn + 1 < tn1) {
      wait_vmcnt<2 * kStores + kTileLoads>();
    } else {
      wait_vmcnt<kStores>();
    }
    const int col = col_of(tn);
#pragma unroll
    for (int u = 0; u < kStores; ++u) {
      asm volatile("" : "+v"(pc[u]));
      Raw8<bf16_t> dv, pv;
      dv.v = make_uint4(rows[u][0], rows[u][1], rows[u][2], rows[u][3]);
      pv.v = make_uint4(pc[u][0], pc[u][1], pc[u][2], pc[u][3]);
      float dp[8], pr[8], ds[8];
      unpack(dv, dp);
      unpack(pv, pr);
      dropout_apply8(g.key, (gidx[u] + col) >> 3, dp);
#pragma unroll
      for (int k = 0; k < 8; ++k) ds[k] = g.scale * (pr[k] * (dp[k] - dot[u]));
      store8(Cbase + static_cast<long long>(row_of(u)) * g.ldc + col, ds);
    }
  };
  // two tiles per trip, so the two sets of P registers swap roles without being copied
  for (int tn = tn0; tn < tn1; tn += 2) {
    tile_step(tn, p0, p1);
    if (tn + 1 < tn1) tile_step(tn + 1, p1, p0);
  }
}

// attention products over whole tiles (grid: tile x matrix in one dimension)
template <bool AK>
hipError_t launch_attn_product(MfmaGemmArgs a, hipStream_t st) {
  constexpr size_t smem = static_cast<size_t>(kStages) * (128 + 128) * kBK * sizeof(bf16_t);
  auto kern = attn_product_kernel<AK>;
  LYNX_RAISE_LDS_LIMIT(kern, smem);
  set_tiles(&a, 128, 128);
  hipLaunchKernelGGL(kern, dim3(a.tiles_m * a.tiles_n * a.nz), dim3(kThreads), smem, st, a);
  return hipGetLastError();
}

// The score-shaped kernels: LDS for the A tile and the B tile / staging area (4 x 64 x 64, the
// larger of the two for short head dimensions).
template <int KD, void (*KERN)(MfmaGemmArgs)>
hipError_t launch_scores(MfmaGemmArgs a, hipStream_t st) {
  constexpr size_t op = static_cast<size_t>(KD / kBK) * 128 * kBK;
  constexpr size_t smem = (op + (op > 4 * 64 * 64 ? op : 4 * 64 * 64)) * sizeof(bf16_t);
  LYNX_RAISE_LDS_LIMIT(KERN, smem);
  a.tiles_m = (a.M + 127) / 128;
  a.tiles_n = a.tiles_m;
  a.run = attn_run(a.tiles_m, a.nz);
  hipLaunchKernelGGL(KERN, dim3(attn_items(a.tiles_m, a.run) * a.nz), dim3(kThreads), smem, st, a);
  return hipGetLastError();
}
hipError_t scores(const MfmaGemmArgs& a, hipStream_t st) {
  const bool whole = a.M % 128 == 0 && (a.K == 64 || a.K == 128);
  if (a.K <= 64)
    return whole ? launch_scores<64, attn_outer_kernel<64, false>>(a, st) : launch_scores<64, attn_outer_kernel<64, true>>(a, st);
  return whole ? launch_scores<128, attn_outer_kernel<128, false>>(a, st) : launch_scores<128, attn_outer_kernel<128, true>>(a, st);
}

}  // namespace

int attention_score_run(int s, int slices) { return attn_run((s + 127) / 128, slices); }

// Attention: score-shaped (S = Q K^T, dPd = dC V^T and dS in its place) and contraction-restricted.
hipError_t gemm_attention(const GemmDesc& d, hipStream_t st) {
  const MfmaGemmArgs a = make_args(d);
  if (d.causal == kCausalOutLower) {
    if (d.epi.kind == kEpiSoftmaxBwd) return launch_scores<128, attn_dscores_kernel>(a, st);
    if (d.K <= 128) return scores(a, st);
    return gemm_ragged(d, nullptr, 0, st);
  }
  // (few tiles: the ragged kernels' 64 x 64 ones)
  if (d.M % 128 || d.N % 128 || is_far(d) || static_cast<long long>(d.M / 128) * (d.N / 128) * a.nz < 256) return gemm_ragged(d, nullptr, 0, st);
  return d.a_sk == 1 ? launch_attn_product<true>(a, st) : launch_attn_product<false>(a, st);
}

}  // namespace lynx
