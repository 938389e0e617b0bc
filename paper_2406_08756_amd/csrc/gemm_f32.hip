// fp32 matrix products on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 sums).
//
// A 32 x 32 x 2 instruction occupies its SIMD's matrix pipe for 64 cycles and reads one register of
// each operand per lane, so the contraction index can run in octets: lane half hb of a fragment holds
// indices 8 c + 4 hb + 0..3 of its row, and instruction j of the octet multiplies element j of both halves.
//
// Contraction slabs travel through an LDS ring of three or four stages filled by direct global -> LDS loads; LDS and
// the loads have time to spare, so no large tile is needed.  What bounds it: the matrix pipe and what is issued between
// its instructions; with buffer loads instead of checked 64-bit pointers and two sums instead of one chain, 1024 tokens,
// 1024 x 4096: 96.5 -> 83.3 us, 4096 x 1024 86.5 -> 78.8; pairs with the longer contraction first 125 -> 111 (QKV), a
// step of that layer 901 -> 821.  Two forms of 16 KB a stage.  64 x 64 per
// workgroup and slabs of 32: a 32 x 32 quarter per wavefront.  32 x 32 per workgroup and slabs of 64, where
// the larger tiles would be fewer than the compute units: each wavefront takes every fourth octet of the
// contraction, and the four sums are added in order at the end.
//
// Sizes are multiples of 8, so chunks of four elements never straddle an edge.  Rows and columns beyond
// the operands repeat the last ones and are not stored, contraction indices beyond K read zeros.
#include "column_partials.h"
#include "device_common.h"
#include "dropout_host.h"
#include "gemm_plans.h"
#include "kernels.h"
#include "mfma_common.h"
#include "pointwise_math.h"

#include <type_traits>

namespace lynx {
namespace {

__device__ const uint4 kZeros = {0u, 0u, 0u, 0u};

// One slab (ROWS x 2048 / ROWS elements, 8 KB) of an operand.
template <int ROWS, bool KMAJOR>
struct SlabF {
  static constexpr int kElems = 2048, kDepth = kElems / ROWS;  // kDepth: contraction indices
  static constexpr int kLoadsPerWave = kElems / 256 / kWaves;  // 1 KB direct loads per wavefront
  static constexpr int kRowChunks = (KMAJOR ? kDepth : ROWS) / 4;  // 16-byte chunks per row of LDS
  // K-major: the chunk permutation spreads 16 consecutive rows, each half the banks wide (kDepth 32) or
  // all of them (64), over all 16-byte columns of the banks.
  __device__ static __forceinline__ int kswz(int row) { return kDepth == 32 ? (row >> 1) & 7 : row & 15; }
  // MN-major: the two lane halves read k-rows four apart, which have to lie in different halves of the
  // banks.  64-wide rows: the columns of every second group of four k-rows are exchanged by halves.
  // 32-wide rows are half the banks themselves: bits 0 and 2 of the k-row trade places.
  __device__ static __forceinline__ int place(int k) { return ROWS == 32 ? (k & ~5) | ((k >> 2) & 1) | ((k & 1) << 2) : k; }
  __device__ static __forceinline__ int mnswz(int k) { return ROWS == 32 ? 0 : ((k >> 2) & 1) << 5; }

  // first element (row mn, contraction index k) of the four that lane `lane` fetches in load j
  __device__ static __forceinline__ int lane_row(int wave, int j, int lane) {  // row of LDS
    return 64 / kRowChunks * (wave + kWaves * j) + lane / kRowChunks;
  }
  __device__ static __forceinline__ int lane_k(int wave, int j, int lane) {
    const int row = lane_row(wave, j, lane);
    return KMAJOR ? ((lane % kRowChunks) ^ kswz(row)) * 4 : place(row);  // (place is its own inverse)
  }
  __device__ static __forceinline__ int lane_mn(int wave, int j, int lane) {
    const int row = lane_row(wave, j, lane);
    return KMAJOR ? row : ((lane % kRowChunks) * 4) ^ mnswz(place(row));
  }
  __device__ static __forceinline__ int lds_offset(int wave, int j) { return (wave + kWaves * j) * 256; }

  // elements 8 c + 4 (lane / 32) + 0..3 of slab row row0 + lane % 32
  __device__ static __forceinline__ void fragment(const float* slab, int row0, int c, int lane, float (&v)[4]) {
    const int r = row0 + (lane & 31), hb = lane >> 5;
    if (KMAJOR) {
      const float32x4_t x = *reinterpret_cast<const float32x4_t*>(slab + r * kDepth + (((2 * c + hb) ^ kswz(r)) << 2));
      v[0] = x[0]; v[1] = x[1]; v[2] = x[2]; v[3] = x[3];
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = 8 * c + 4 * hb + j;
        v[j] = slab[place(k) * ROWS + (r ^ mnswz(k))];
      }
    }
  }
};

constexpr int kLarge = 64, kSmall = 32;   // tile sides
constexpr long long kFarStride = 1ll << 23;  // row strides (elements) from which on 32 bits may not hold a load's offset in bytes
// Ring stages of 16 KB.  64 x 64: three, so that three workgroups share a compute unit and cover each other's barriers,
// fills and store passes; with four (two workgroups) a step of 1024 tokens of h 1024 takes 808 us where this takes 786, with
// two (five workgroups, one slab ahead) 899.  Four where a third does not help: deep_ring().  32 x 32: four; such
// launches do not fill the chip, and a layer of 256 tokens of h 256 takes 141.2 us this way, 142.5 with three.
constexpr int kShallow = 3, kDeep = 4;
constexpr int kPitchPad = 4;              // floats: keeps the 16-byte accesses of the staged tile off each other's banks
template <int S> constexpr size_t kLdsBytes = S * 2 * 2048 * sizeof(float);
static_assert(kLdsBytes<kDeep> >= kWaves * 32 * (kSmall + kPitchPad) * sizeof(float) &&
                  kLdsBytes<kShallow> >= kLarge * (kLarge + kPitchPad) * sizeof(float),
              "the staged tile fits the ring");

// Where a tile lies and what it contracts over.
struct F32Tile {
  int tm, m0, n0, k_begin, k_end;
  const float *A, *B;
  float* C;
};
template <int BM>
__device__ __forceinline__ F32Tile locate(const GemmDesc& d, int block_x, int block_z) {
  F32Tile t;
  const int tiles_n = (d.N + BM - 1) / BM;
  int tn;
  if (d.causal == kCausalOutLower) {          // square output, tiles on or below the diagonal only
    t.tm = static_cast<int>((sqrtf(8.0f * static_cast<float>(block_x) + 1.0f) - 1.0f) * 0.5f);
    while (t.tm * (t.tm + 1) / 2 > block_x) --t.tm;
    while ((t.tm + 1) * (t.tm + 2) / 2 <= block_x) ++t.tm;
    tn = block_x - t.tm * (t.tm + 1) / 2;
  } else {
    t.tm = block_x / tiles_n;
    tn = block_x - t.tm * tiles_n;
    if (d.causal == kCausalKLeM) t.tm = (d.M + BM - 1) / BM - 1 - t.tm;   // longest contraction first
  }
  t.m0 = t.tm * BM;
  t.n0 = tn * BM;
  // (the seq x seq operands are zero beyond the diagonal up to the next multiple of 128)
  t.k_begin = d.causal == kCausalKGeM ? t.m0 : 0;
  t.k_end = d.causal == kCausalKLeM ? min(d.K, t.m0 + BM) : d.K;
  const int z1 = block_z / d.nz2, z2 = block_z - z1 * d.nz2;
  t.A = static_cast<const float*>(d.A) + z1 * d.a_sz1 + z2 * d.a_sz2;
  t.B = static_cast<const float*>(d.B) + z1 * d.b_sz1 + z2 * d.b_sz2;
  t.C = static_cast<float*>(d.C) + z1 * d.c_sz1 + z2 * d.c_sz2;
  return t;
}

// The store pass.  acc[r] is the element n = 8 (r / 4) + 4 (lane / 32) + r % 4, m = lane % 32 of the
// wavefront's 32 x 32: through LDS into octets of a row, which take bias and epilogue.
template <int BM>
__device__ __forceinline__ void store_tile(const GemmDesc& d, const DropoutKey& key, const F32Tile& t, float* smem,
                                           const floatx16_t& acc, int wave, int lane) {
  constexpr bool kSum = BM == kSmall;        // the four wavefronts hold parts of the same 32 x 32
  constexpr int kPitch = BM + kPitchPad, kPart = 32 * kPitch;
  const int tid = threadIdx.x;
  float* stage = smem + (kSum ? wave * kPart : (wave >> 1) * 32 * kPitch + (wave & 1) * 32);
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<float4*>(stage + (lane & 31) * kPitch + 8 * q + 4 * (lane >> 5)) =
        make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
  __syncthreads();
  constexpr int kRowOctets = BM / 8, kRowsAtOnce = kThreads / kRowOctets;
  const int lr = tid / kRowOctets, lc = tid % kRowOctets;
  const int n = t.n0 + lc * 8;
  const bool col_in = n < d.N;
  float bias[8] = {}, colacc[8] = {};
  if (d.bias != nullptr && col_in) load8(static_cast<const float*>(d.bias) + n, bias);
  if (d.epi.kind == kEpiBiasDropoutAdd && col_in) load8(static_cast<const float*>(d.epi.vec) + n, bias);
#pragma unroll
  for (int r0 = 0; r0 < BM; r0 += kRowsAtOnce) {
    const int r = r0 + lr, m = t.m0 + r;
    if (r >= BM || m >= d.M || !col_in) continue;
    float v[8];
    load8(smem + r * kPitch + lc * 8, v);
    if (kSum) {
#pragma unroll
      for (int w = 1; w < kWaves; ++w) {
        float p[8];
        load8(smem + w * kPart + r * kPitch + lc * 8, p);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] += p[i];
      }
    }
    float* c = t.C + m * d.c_sm + n;
    if (d.epi.kind == kEpiNone || d.epi.kind == kEpiGelu) {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] += bias[i];
      if (d.epi.kind == kEpiGelu) {
        if (d.epi.plain != nullptr) store8(static_cast<float*>(d.epi.plain) + m * d.c_sm + n, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = gelu_f(v[i]);
      }
      store8(c, v);
    } else {
      float x[8], o[8];
      load8(static_cast<const float*>(d.epi.aux) + m * d.epi.aux_ld + n, x);
      if (d.epi.kind == kEpiBiasDropoutAdd) {
        if (d.epi.plain != nullptr) store8(static_cast<float*>(d.epi.plain) + m * d.c_sm + n, v);
        bias_dropout_add8(v, bias, x, key, (static_cast<uint64_t>(m) * static_cast<uint64_t>(d.N) + n) >> 3, o);
      } else {
        gelu_bwd8<float>(v, x, o);
#pragma unroll
        for (int i = 0; i < 8; ++i) colacc[i] += o[i];
      }
      store8(c, o);
    }
  }
  if (d.epi.kind == kEpiGeluBwd) {
    // column sums of the tile: over the rows of a wavefront, then over the wavefronts in order
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int o = kRowOctets; o < kWave; o <<= 1) colacc[i] += __shfl_xor(colacc[i], o, kWave);
    __syncthreads();
    if (lane < kRowOctets)
#pragma unroll
      for (int i = 0; i < 8; ++i) smem[wave * BM + lane * 8 + i] = colacc[i];
    __syncthreads();
    if (tid < BM && t.n0 + tid < d.N)
      d.epi.colsum_partial[static_cast<long long>(t.tm) * d.N + t.n0 + tid] =
          (smem[tid] + smem[BM + tid]) + (smem[2 * BM + tid] + smem[3 * BM + tid]);
  }
}

template <bool AK, bool BK, int BM, int S>
__device__ __forceinline__ void f32_tile(const GemmDesc& d, const DropoutKey& key, int block_x, int block_z) {
  constexpr int kAhead = S - 1;
  using SA = SlabF<BM, AK>;
  using SB = SlabF<BM, BK>;
  constexpr bool kShareTile = BM == kSmall;  // the wavefronts divide the contraction, not the tile
  constexpr int kSlab = SA::kDepth;
  constexpr int kOctets = kSlab / 8 / (kShareTile ? kWaves : 1);  // per wavefront and slab
  constexpr int kStage = SA::kElems + SB::kElems;
  constexpr int kLoads = SA::kLoadsPerWave + SB::kLoadsPerWave;
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  float* smem = reinterpret_cast<float*>(smem_raw);
  const F32Tile t = locate<BM>(d, block_x, block_z);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = kShareTile ? 0 : (wave >> 1) * 32, wn0 = kShareTile ? 0 : (wave & 1) * 32;

  const long long lda = AK ? d.a_sm : d.a_sk, ldb = BK ? d.b_sn : d.b_sk;
  const float* ga[SA::kLoadsPerWave];
  const float* gb[SB::kLoadsPerWave];
#pragma unroll
  for (int j = 0; j < SA::kLoadsPerWave; ++j) {
    const long long mn = min(t.m0 + SA::lane_mn(wave, j, lane), d.M - (AK ? 1 : 4)), k = t.k_begin + SA::lane_k(wave, j, lane);
    ga[j] = t.A + (AK ? mn * lda + k : k * lda + mn);
  }
#pragma unroll
  for (int j = 0; j < SB::kLoadsPerWave; ++j) {
    const long long mn = min(t.n0 + SB::lane_mn(wave, j, lane), d.N - (BK ? 1 : 4)), k = t.k_begin + SB::lane_k(wave, j, lane);
    gb[j] = t.B + (BK ? mn * ldb + k : k * ldb + mn);
  }
  const long long a_step = AK ? kSlab : kSlab * lda, b_step = BK ? kSlab : kSlab * ldb;
  // Whole slabs: buffer loads from the operand's tile corner, in scalar registers, with 32-bit lane offsets, so that no
  // address arithmetic stands between the matrix instructions.  (Strides of kFarStride and more: pointers throughout.)
  const float* const corner_a = t.A + (AK ? t.m0 * lda + t.k_begin : t.k_begin * lda + t.m0);
  const float* const corner_b = t.B + (BK ? t.n0 * ldb + t.k_begin : t.k_begin * ldb + t.n0);
  uint32_t oa[SA::kLoadsPerWave], ob[SB::kLoadsPerWave];
#pragma unroll
  for (int j = 0; j < SA::kLoadsPerWave; ++j) oa[j] = static_cast<uint32_t>(4 * (ga[j] - corner_a));
#pragma unroll
  for (int j = 0; j < SB::kLoadsPerWave; ++j) ob[j] = static_cast<uint32_t>(4 * (gb[j] - corner_b));
  const int nk = (t.k_end - t.k_begin + kSlab - 1) / kSlab;
  const int k_rem = (t.k_end - t.k_begin) % kSlab;
  const int tail = k_rem != 0 ? nk - 1 : -1;  // the slab that reaches beyond the contraction range
  auto issue_load = [&](auto steady_tag, int kt, int j) {
    float* s = smem + (kt % S) * kStage;
    if constexpr (decltype(steady_tag)::value) {
      const bool of_a = j < SA::kLoadsPerWave;
      const int jb = j - SA::kLoadsPerWave;
      buffer_load_to_lds(of_a ? corner_a + kt * a_step : corner_b + kt * b_step, of_a ? oa[j] : ob[jb],
                         reinterpret_cast<bf16_t*>(of_a ? s + SA::lds_offset(wave, j) : s + SA::kElems + SB::lds_offset(wave, jb)));
      return;
    }
    if (j < SA::kLoadsPerWave) {
      const float* from = ga[j] + kt * a_step;
      if (kt == tail && SA::lane_k(wave, j, lane) >= k_rem) from = reinterpret_cast<const float*>(&kZeros);
      __builtin_amdgcn_global_load_lds((global_void_ptr)(from), (lds_void_ptr)(s + SA::lds_offset(wave, j)), 16, 0, 0);
    } else {
      const int jb = j - SA::kLoadsPerWave;
      const float* from = gb[jb] + kt * b_step;
      if (kt == tail && SB::lane_k(wave, jb, lane) >= k_rem) from = reinterpret_cast<const float*>(&kZeros);
      __builtin_amdgcn_global_load_lds((global_void_ptr)(from), (lds_void_ptr)(s + SA::kElems + SB::lds_offset(wave, jb)), 16, 0, 0);
    }
  };

  // two sums, of every second index: consecutive instructions do not wait for each other
  floatx16_t acc[2];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][r] = acc[1][r] = 0.f;
#pragma unroll
  for (int i = 0; i < kAhead; ++i)
    if (i < nk)
#pragma unroll
      for (int j = 0; j < kLoads; ++j) issue_load(std::false_type{}, i, j);
  wait_slabs<kLoads, kAhead - 1>(nk - 1);
  block_barrier();
  // A slab is kOctets octets of four instructions.  Over the first half of them the octets of the second
  // half are read and the ring stage that was finished before the last barrier is refilled; then [next
  // slab landed?] [barrier]; over the second half the next slab's first octets are read.
  float fa[kOctets][4], fb[kOctets][4];
  auto read = [&](const float* stage, int f, int i0) {   // f: A and B of octets i0, i0 + 1, ... in turn
    const int i = i0 + (f >> 1), c = kShareTile ? wave + kWaves * i : i;
    if ((f & 1) == 0) SA::fragment(stage, wm0, c, lane, fa[i]);
    else SB::fragment(stage + SA::kElems, wn0, c, lane, fb[i]);
  };
#pragma unroll
  for (int f = 0; f < kOctets; ++f) read(smem, f, 0);
  constexpr int kHalf = 2 * kOctets;                         // instructions of half a slab
  constexpr int kPer = (kOctets + kLoads + kHalf - 1) / kHalf;  // side operations per instruction
  auto slab_step = [&](int kt, auto steady_tag) {
    constexpr bool steady = decltype(steady_tag)::value;
    const float* cur = smem + (kt % S) * kStage;
    const float* next = smem + ((kt + 1) % S) * kStage;
    const bool refill = steady || kt + kAhead < nk, more = steady || kt + 1 < nk;
#pragma unroll
    for (int m = 0; m < 2 * kHalf; ++m) {
      if (m == kHalf) {
        if (steady) wait_vmcnt<(kAhead - 1) * kLoads>();
        else wait_slabs<kLoads, kAhead - 1>(nk - 2 - kt);
        block_barrier();
      }
      acc[m & 1] = __builtin_amdgcn_mfma_f32_32x32x2f32(fb[m >> 2][m & 3], fa[m >> 2][m & 3], acc[m & 1], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int op = (m % kHalf) * kPer + u;
        if (m >= kHalf) {
          if (op < kOctets && more) read(next, op, 0);
        } else if (op < kOctets) {
          read(cur, op, kOctets / 2);
        } else if (op < kOctets + kLoads && refill) {
          issue_load(steady_tag, kt + kAhead, op - kOctets);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int kt = 0;
  const int whole = lda >= kFarStride || ldb >= kFarStride ? 0 : (tail < 0 ? nk : tail);
  for (; kt + kAhead < whole; ++kt) slab_step(kt, std::true_type{});
  for (; kt < nk; ++kt) slab_step(kt, std::false_type{});
  block_barrier();
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[0][r] += acc[1][r];
  store_tile<BM>(d, key, t, smem, acc[0], wave, lane);
}

template <bool AK, bool BK, int BM, int S>
__global__ void __launch_bounds__(kThreads) gemm_f32_kernel(GemmDesc d, DropoutKey key) {
  f32_tile<AK, BK, BM, S>(d, key, blockIdx.x, blockIdx.y);
}

// Input and weight gradient of a linear layer in one launch, so that together they fill the chip: the first n_first
// workgroups belong to the one with the longer contraction, the others fill what it leaves idle.
template <int BM, int S>
__device__ __forceinline__ void f32_pair_tile(const GemmDesc& wgrad, const GemmDesc& dgrad, const DropoutKey& key, int n_first, int dgrad_first, int x) {
  const int tile = x < n_first ? x : x - n_first;
  if ((x < n_first) != (dgrad_first != 0)) f32_tile<false, false, BM, S>(wgrad, key, tile, 0);
  else f32_tile<true, false, BM, S>(dgrad, key, tile, 0);
}
template <int BM, int S>
__global__ void __launch_bounds__(kThreads) gemm_f32_pair_kernel(GemmDesc wgrad, GemmDesc dgrad, DropoutKey key, int n_first, int dgrad_first) {
  f32_pair_tile<BM, S>(wgrad, dgrad, key, n_first, dgrad_first, blockIdx.x);
}
// ... and a column sum besides, in workgroups between them.  The rows that the guest has in flight raise the registers of all
// (VGPRs and AGPRs) from 100 (64 x 64) and 84 to 140; three wavefronts per SIMD, as the ring of 64 x 64 tiles is made
// for, may have 168.  (No bound says so: given one, the compiler spends 128 and waits between the guest's loads.)
template <int BM, int S>
__global__ void __launch_bounds__(kThreads)
gemm_f32_pair_guest_kernel(GemmDesc wgrad, GemmDesc dgrad, DropoutKey key, int n_first, int dgrad_first, ColumnPartials guest) {
  const int x = static_cast<int>(blockIdx.x);
  if (x >= guest.first && x < guest.end) column_partials<float>(guest, (x - guest.first) * kWaves + static_cast<int>(threadIdx.x) / kWave);
  else f32_pair_tile<BM, S>(wgrad, dgrad, key, n_first, dgrad_first, x < guest.first ? x : x - (guest.end - guest.first));
}

// Two products of attention that do not need each other (batched alike) in one launch: few tiles each, and a launch of
// either leaves half of the chip's wavefronts out.  Workgroups of both in turn as long as both have some.
template <bool AK1, bool BK1, bool AK2, bool BK2, int BM, int S>
__global__ void __launch_bounds__(kThreads) gemm_f32_two_kernel(GemmDesc d1, GemmDesc d2, int n1, int n2) {
  const int x = static_cast<int>(blockIdx.x), both = 2 * min(n1, n2);
  const bool second = x < both ? (x & 1) != 0 : n2 > n1;
  const int tile = x < both ? x >> 1 : x - both / 2;
  if (second) f32_tile<AK2, BK2, BM, S>(d2, DropoutKey{}, tile, blockIdx.y);
  else f32_tile<AK1, BK1, BM, S>(d1, DropoutKey{}, tile, blockIdx.y);
}

long long tiles(const GemmDesc& d, int bm) {
  const long long tm = (d.M + bm - 1) / bm, tn = (d.N + bm - 1) / bm;
  return d.causal == kCausalOutLower ? tm * (tm + 1) / 2 : tm * tn;
}

// 64 x 64 tiles take 1.15 times less per multiplication where they fill the chip (4096^3: 1207 against 1354 us,
// 114 and 101 TFLOP/s; the vector-ALU kernel before these ran at 20); 32 x 32 where whole rounds of the
// larger ones over the 256 compute units would cost more than that (256 x 256 x 1024: 24.1 against 8.5 us,
// 85 before; 1024^3, one 64 x 64 tile per unit: 25.3 against 24.7).
bool small_tiles(long long tiles64) { return (tiles64 + 255) / 256 * 256 > 1.15 * tiles64; }

// Four stages in 64 x 64 tiles, with three / four us each: one workgroup per unit, which nothing but its own loads can
// cover (FC2's forward, 256 workgroups: 1024 tokens of h 1024, f 4096 84 / 79, f 2048 45 / 43, 256 tokens 26.1 / 25.6; dQ and dK of
// 30 slices of s = 72, 240 workgroups, 7.3 / 6.4; with two per unit nothing is lost by three).
bool deep_ring(long long workgroups) { return workgroups <= 256; }
// Pairs, whose longer contraction comes first.  Four stages where
//  - it alone takes 0.6 of the time that an even share of all does: its workgroups are done last, so what counts is their own
//    time.  FC1's gradients of 192, 256, 384 and 512 tokens of h 1280 (2.1, 1.6, 1.1 and 0.8 of it) 100 / 94, 103 / 99, 116 / 108 and
//    129 / 122, of 512 of h 768 (0.67) 69 / 63; at 0.5 FC1's of 1024 of h 1024 139 / 151, QKV's there 104 / 107;
//  - all are placed at once, the third on units that have two long ones, where of two at a time the short ones would all go to
//    units with a short one: FC1's of 1152 tokens of h 960, f 1920 (270 and 450 workgroups, 1920 and 1152 long) 84 / 75, a pass of 432 of
//    h 640 (280 and 400, 640 and 432) 273 / 268; but 512 of h 640 (320 and 400) 37 / 44;
//  - contractions are of much the same length and more than half of the units have a fourth, and none a fifth, which of three
//    at a time runs alone: FC2's of 1024 tokens of h 1024, f 2048 88 / 77, QKV's of 1856 of h 872, 980 workgroups, 157 / 146; but 896
//    of them, FC2's of 768 of h 1024, f 2048, 61 / 66.
// With more of them, three: FC2's of 256 tokens of h 1280 62 / 70, of 512 117 / 125, FC1's of 1024 of h 1024 139 / 151.
bool deep_ring_pair(const GemmDesc& a, long long n_a, const GemmDesc& b, long long n_b) {
  const bool a_longer = a.K > b.K;
  const long long even = (n_a * a.K + n_b * b.K) / 256, n = n_a + n_b, n_long = a_longer ? n_a : n_b;
  const long long longer = a_longer ? a.K : b.K, shorter = a_longer ? b.K : a.K;
  if (5 * longer > 3 * even) return true;
  if (n > 768) return n > 896 && n <= 1024 && 2 * longer <= 3 * shorter;
  if (n <= 512 || n_long <= 256 || n - 512 > 512 - n_long) return false;
  const long long most = longer + 2 * shorter > 2 * longer ? longer + 2 * shorter : 2 * longer;  // of one unit, two at a time
  return 16 * most < 15 * (2 * longer + shorter);
}
}  // namespace

F32Choice gemm_f32_choice(const GemmDesc& d) {
  if (small_tiles(tiles(d, kLarge) * d.nz1 * d.nz2)) return {kSmall, kDeep};
  return {kLarge, deep_ring(tiles(d, kLarge) * d.nz1 * d.nz2) ? kDeep : kShallow};
}
F32Choice gemm_f32_pair_choice(const GemmDesc& dgrad, const GemmDesc& wgrad) {
  const long long n_d = tiles(dgrad, kLarge), n_w = tiles(wgrad, kLarge);
  if (small_tiles(n_d + n_w)) return {kSmall, kDeep};
  return {kLarge, deep_ring_pair(dgrad, n_d, wgrad, n_w) ? kDeep : kShallow};
}

namespace {
DropoutKey epilogue_key(const GemmDesc& d) {
  return d.epi.kind == kEpiBiasDropoutAdd ? make_dropout_key(d.epi.dp, d.epi.site) : DropoutKey{};
}

template <bool AK, bool BK, int BM, int S>
hipError_t launch(const GemmDesc& d, hipStream_t st) {
  hipLaunchKernelGGL((gemm_f32_kernel<AK, BK, BM, S>), dim3(static_cast<unsigned>(tiles(d, BM)), d.nz1 * d.nz2), dim3(kThreads),
                     kLdsBytes<S>, st, d, epilogue_key(d));
  return hipGetLastError();
}
template <bool AK, bool BK>
hipError_t launch(const GemmDesc& d, hipStream_t st) {
  const F32Choice c = gemm_f32_choice(d);
  if (c.tile == kSmall) return launch<AK, BK, kSmall, kDeep>(d, st);
  if (c.stages == kDeep) return launch<AK, BK, kLarge, kDeep>(d, st);
  return launch<AK, BK, kLarge, kShallow>(d, st);
}

template <bool AK1, bool BK1, bool AK2, bool BK2, int BM, int S>
hipError_t launch_two(const GemmDesc& a, const GemmDesc& b, hipStream_t st) {
  const int n1 = static_cast<int>(tiles(a, BM)), n2 = static_cast<int>(tiles(b, BM));
  hipLaunchKernelGGL((gemm_f32_two_kernel<AK1, BK1, AK2, BK2, BM, S>), dim3(n1 + n2, a.nz1 * a.nz2), dim3(kThreads), kLdsBytes<S>, st, a, b, n1, n2);
  return hipGetLastError();
}
template <bool AK1, bool BK1, bool AK2, bool BK2>
hipError_t launch_two(const GemmDesc& a, const GemmDesc& b, hipStream_t st) {
  const long long workgroups = (tiles(a, kLarge) + tiles(b, kLarge)) * a.nz1 * a.nz2;
  if (small_tiles(workgroups)) return launch_two<AK1, BK1, AK2, BK2, kSmall, kDeep>(a, b, st);
  if (deep_ring(workgroups)) return launch_two<AK1, BK1, AK2, BK2, kLarge, kDeep>(a, b, st);
  return launch_two<AK1, BK1, AK2, BK2, kLarge, kShallow>(a, b, st);
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

bool gemm_f32_supported(const GemmDesc& d) {
  if (d.M % 8 || d.N % 8 || d.K % 8 || d.M <= 0 || d.N <= 0 || d.K <= 0) return false;
  if (d.causal == kCausalOutLower && d.M != d.N) return false;
  const bool a_k = d.a_sk == 1, b_k = d.b_sk == 1;
  if ((!a_k && d.a_sm != 1) || (!b_k && d.b_sn != 1) || (!a_k && b_k)) return false;
  if ((a_k ? d.a_sm : d.a_sk) % 4 || (b_k ? d.b_sn : d.b_sk) % 4 || d.c_sm % 4) return false;
  if (d.a_sz1 % 4 || d.a_sz2 % 4 || d.b_sz1 % 4 || d.b_sz2 % 4 || d.c_sz1 % 4 || d.c_sz2 % 4) return false;
  if (!aligned16(d.A) || !aligned16(d.B) || !aligned16(d.C) || !aligned16(d.bias)) return false;
  switch (d.epi.kind) {
    case kEpiNone: return true;
    case kEpiGelu: return d.causal == kCausalNone && d.nz1 * d.nz2 == 1 && aligned16(d.epi.plain);
    case kEpiBiasDropoutAdd:
      return d.causal == kCausalNone && d.nz1 * d.nz2 == 1 && d.bias == nullptr && d.epi.aux != nullptr &&
             aligned16(d.epi.aux) && d.epi.aux_ld % 4 == 0 && d.epi.vec != nullptr && aligned16(d.epi.vec) &&
             aligned16(d.epi.plain);
    case kEpiGeluBwd:
      return d.causal == kCausalNone && d.nz1 * d.nz2 == 1 && d.bias == nullptr && d.epi.aux != nullptr &&
             aligned16(d.epi.aux) && d.epi.aux_ld % 4 == 0 && d.epi.colsum_partial != nullptr && d.epi.colsum_out != nullptr;
  }
  return false;
}

hipError_t gemm_f32(const GemmDesc& d, hipStream_t st) {
  if (d.epi.kind == kEpiGeluBwd) return hipErrorInvalidValue;  // in a pair only
  if (d.a_sk != 1) return launch<false, false>(d, st);
  return d.b_sk == 1 ? launch<true, true>(d, st) : launch<true, false>(d, st);
}

hipError_t gemm_f32_two(const GemmDesc& a, const GemmDesc& b, hipStream_t st) {
  if (a.nz1 != b.nz1 || a.nz2 != b.nz2 || a.epi.kind != kEpiNone || b.epi.kind != kEpiNone || a.a_sk != 1 || b.a_sk == 1)
    return hipErrorInvalidValue;
  return a.b_sk == 1 ? launch_two<true, true, false, false>(a, b, st) : launch_two<true, false, false, false>(a, b, st);
}

size_t gemm_f32_pair_colsum_bytes(const GemmDesc& dgrad, const GemmDesc& wgrad) {
  const int bm = gemm_f32_pair_choice(dgrad, wgrad).tile;
  return static_cast<size_t>((dgrad.M + bm - 1) / bm) * dgrad.N * sizeof(float);
}

hipError_t gemm_f32_pair(const GemmDesc& dgrad, const GemmDesc& wgrad, const ColumnSumInput* in, ColumnSums* sums, hipStream_t st) {
  const F32Choice c = gemm_f32_pair_choice(dgrad, wgrad);
  const int bm = c.tile;
  const int n_w = static_cast<int>(tiles(wgrad, bm)), n_d = static_cast<int>(tiles(dgrad, bm));
  const bool dgrad_first = dgrad.K > wgrad.K;
  const int n_first = dgrad_first ? n_d : n_w;
  auto launch_pair = [&](auto bm_tag, auto stages_tag) {
    constexpr int BM = decltype(bm_tag)::value, S = decltype(stages_tag)::value;
    if (in != nullptr) {
      const ColumnPartials guest = guest_partials(*in, n_first, n_w + n_d, kWaves);
      hipLaunchKernelGGL((gemm_f32_pair_guest_kernel<BM, S>), dim3(n_w + n_d + guest.end - guest.first), dim3(kThreads), kLdsBytes<S>, st, wgrad, dgrad,
                         DropoutKey{}, n_first, dgrad_first ? 1 : 0, guest);
    } else {
      hipLaunchKernelGGL((gemm_f32_pair_kernel<BM, S>), dim3(n_w + n_d), dim3(kThreads), kLdsBytes<S>, st, wgrad, dgrad, DropoutKey{},
                         n_first, dgrad_first ? 1 : 0);
    }
  };
  constexpr std::integral_constant<int, kShallow> shallow{};
  constexpr std::integral_constant<int, kDeep> deep{};
  if (c.tile == kSmall) launch_pair(std::integral_constant<int, kSmall>{}, deep);
  else if (c.stages == kDeep) launch_pair(std::integral_constant<int, kLarge>{}, deep);
  else launch_pair(std::integral_constant<int, kLarge>{}, shallow);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && in != nullptr) e = sums->add(in->part, in->out, (in->rows + kPartialRows - 1) / kPartialRows, in->cols);
  if (e != hipSuccess || dgrad.epi.kind != kEpiGeluBwd) return e;
  return sums->add(dgrad.epi.colsum_partial, dgrad.epi.colsum_out, (dgrad.M + bm - 1) / bm, dgrad.N);
}

}  // namespace lynx
