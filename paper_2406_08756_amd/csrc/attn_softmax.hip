// Operators 3 to 5 in one launch (bf16, s <= 2048, head dimension <= 128): S = Q K^T, P = softmax(S / sqrt(d)) over
// j <= i, Pd = dropout(P).  S, P and Pd are written as far as somebody wants them; the bits of each are those of
// the kernels that form them one after the other (attn_outer_kernel, softmax_dropout_fwd_kernel).
//
// What it saves is S's way through memory, a write and a read of b a s^2 values, and a launch.  What bounds it: the
// vector ALU (exponentials, the dropout generator, rounding), about 90 cycles per 64 values, 32 more where exponentials
// are formed twice (below), then its loads of K and its stores.  Separate kernels and this one, us: 40 slices of
// s = 2048, d = 128, Pd alone 142 and 104, P and Pd 151 and 118; 64 slices 208 and 158, 250 and 187; 128 of 1024, d = 64,
// S, P and Pd 128 and 98; 100 of 1000, d = 64, Pd 94 and 64, P and Pd 109 and 78; 8 of 384, a forward pass 43.8 and 41.2.
//
// A workgroup of WAVES wavefronts owns 32 rows of one slice.  Wavefront w takes the 64-column blocks w, w + WAVES, ...
// up to the diagonal: it loads its rows of K into LDS by itself, 8 KB at a time, multiplies (products formed
// transposed, so a lane holds 16 columns of one row per 32 x 32 tile, four consecutive ones at a time) and keeps the
// rounded scores in registers, 16 per block.  Then the row maxima go round the wavefronts through LDS, then the
// block sums (the canonical order of attn_math.h, whose group of 4 is a lane's four columns and whose tree of 8 a
// lane's block), and every wavefront normalises its blocks, passes them through LDS into whole rows and stores those,
// one dropout call per 8 columns.  At most two blocks per wavefront, of four wavefronts where s <= 512 and of eight beyond;
// of rows longer than 1024 up to four blocks, whose exponentials are formed again for the normalisation instead of
// being kept: at most 128 registers (forms of ragged shapes with four blocks, and two of the gradient with two, spill one or
// two more), and four wavefronts per SIMD cover each other's loads, transcendentals and stores.
// (Four wavefronts of up to eight blocks, two per SIMD, 40 slices of s = 2048: 148 us with P, 119 without.)
#include <mutex>

#include "attn_math.h"
#include "dropout_host.h"
#include "gemm_launch.h"

namespace lynx {
namespace {

constexpr int kRowsOfBlock = 32, kColsOfBlock = 64;
constexpr int kMaxSeq = 2048;
constexpr int kMaxBlocks = kMaxSeq / kColsOfBlock;
constexpr int kStepElems = 4096;  // K of one step of one wavefront: 64 rows of head dimension 64, or 32 of 128

struct ScoresSoftmaxArgs {
  const bf16_t* q; const bf16_t* k;
  long long ld;
  bf16_t* S; bf16_t* P; bf16_t* Pd;  // nullable
  int s, d, a, nz, row_blocks;
  int global_heads, head0;
  float scale;
  DropoutKey key;
  int stream_s, stream_p;  // streaming stores
};

// One 16-byte store per lane, streaming or not.
__device__ __forceinline__ void store_row(const RowBuffer& b, uint32_t offset, uintx4_t v, bool streaming) {
  if (streaming) row_buffer_store_streaming(b, offset, v);
  else row_buffer_store(b, offset, v);
}

// Slab sl (64 of the head dimension) of the rows from row0 on of a [s, d] operand with row stride ld.  Whole ones through
// buffer loads: eight rows each, whose corner is uniform and whose lane offsets repeat every second load (the
// permutation of Slab has period 16 rows).
template <typename SL, int KD, bool RAGGED>
__device__ __forceinline__ void load_rows(const bf16_t* base, long long ld, int s, int d, int row0, int sl, bf16_t* to, int lane) {
  if (!RAGGED || (d == KD && row0 + 8 * SL::kLoadsPerWave <= s)) {
    uint32_t offset[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
      offset[j] = static_cast<uint32_t>(lane >> 3) * static_cast<uint32_t>(2 * ld) + 2 * static_cast<uint32_t>(SL::lane_k(0, j, lane));
#pragma unroll
    for (int j = 0; j < SL::kLoadsPerWave; ++j)
      buffer_load_to_lds(base + (row0 + 8 * j) * ld + sl * 64, offset[j & 1], to + SL::lds_offset(0, j));
    return;
  }
#pragma unroll
  for (int j = 0; j < SL::kLoadsPerWave; ++j) {
    const int row = min(row0 + SL::lane_mn(0, j, lane), s - 1);
    const int kk = sl * 64 + SL::lane_k(0, j, lane);
    const bf16_t* from = base + row * ld + kk;
    if (kk >= d) from = reinterpret_cast<const bf16_t*>(&kZeroChunk);
    __builtin_amdgcn_global_load_lds((global_void_ptr)(from), (lds_void_ptr)(to + SL::lds_offset(0, j)), 16, 0, 0);
  }
}

// NBW: most blocks per wavefront.
template <int KD, bool RAGGED, int WAVES, int NBW>
__global__ void __launch_bounds__(WAVES * kWave, WAVES == 8 ? 4 : 3) attn_scores_softmax_kernel(ScoresSoftmaxArgs g) {
  constexpr int kSlabs = KD / 64;
  constexpr int kStepCols = kStepElems / KD, kSteps = kColsOfBlock / kStepCols;  // of a block
  using SQ = Slab<kRowsOfBlock, true, 64, 1>;
  using SK = Slab<kStepCols, true, 64, 1>;
  constexpr bool kKeep = NBW <= 2;  // exponentials stay in registers
  // longest rows first; slice z on XCD z % 8 where the slices are a multiple of 8
  const int rb = g.row_blocks - 1 - static_cast<int>(blockIdx.x) / g.nz;
  const int bz = static_cast<int>(blockIdx.x) % g.nz;
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* sQ = reinterpret_cast<bf16_t*>(smem_raw);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  bf16_t* sK = sQ + kSlabs * SQ::kElems + wave * kStepElems;  // this wavefront's; later its staging area
  float* row_max = reinterpret_cast<float*>(sQ + kSlabs * SQ::kElems + WAVES * kStepElems);  // [WAVES][32]
  float* block_sum = row_max + WAVES * kRowsOfBlock;                                       // [kMaxBlocks][32]

  const int z1 = bz / g.a, z2 = bz - z1 * g.a;
  const long long slice = z1 * static_cast<long long>(g.s) * g.ld + static_cast<long long>(z2) * g.d;
  const bf16_t* q = g.q + slice;
  const bf16_t* k = g.k + slice;
  const int r0 = rb * kRowsOfBlock;
  const int rows_in = RAGGED ? min(kRowsOfBlock, g.s - r0) : kRowsOfBlock;
  const int active = (r0 + rows_in - 1) / kColsOfBlock + 1;              // blocks up to the diagonal
  const int padded = min(g.s, (r0 + rows_in + 127) / 128 * 128);         // columns written (zeros beyond the diagonal)
  const int blocks = (padded + kColsOfBlock - 1) / kColsOfBlock;

  auto load_k = [&](int col) {
#pragma unroll
    for (int sl = 0; sl < kSlabs; ++sl) load_rows<SK, KD, RAGGED>(k, g.ld, g.s, g.d, col, sl, sK + sl * SK::kElems, lane);
  };
  if (wave < kSlabs) load_rows<SQ, KD, RAGGED>(q, g.ld, g.s, g.d, r0, wave, sQ + wave * SQ::kElems, lane);
  if (wave < active) load_k(wave * kColsOfBlock);
  wait_vmcnt<0>();
  block_barrier();

  const int my_row = r0 + (lane & 31), half = lane >> 5;
  // Staging, 32 rows of 64 columns, and the row layout it is read back in.  Two rows are as wide as the LDS banks: the
  // 16-byte chunk is permuted by bits 1 to 3 of the row, the half of a chunk by bit 4, so that 32 rows' writes of 8
  // bytes fall into different banks (the reader swaps the halves of rows 16 to 31 back).
  const int lr = lane >> 3, lc = lane & 7;
  bf16_t* const stage_to = sK + (lane & 31) * kColsOfBlock + 4 * (half ^ ((lane >> 4) & 1));
  auto stage_write = [&](int i, int qd, uint2 v) {
    *reinterpret_cast<uint2*>(stage_to + (((4 * i + qd) ^ ((lane >> 1) & 7)) << 3)) = v;
  };
  auto stage_read = [&](int u) {
    const int row = u * 8 + lr;
    const uintx4_t v = *reinterpret_cast<const uintx4_t*>(sK + row * kColsOfBlock + ((lc ^ ((row >> 1) & 7)) << 3));
    return u < 2 ? v : uintx4_t{v[2], v[3], v[0], v[1]};
  };
  const long long out0 = (static_cast<long long>(bz) * g.s + r0) * g.s;
  const uint32_t row_bytes = 2u * static_cast<uint32_t>(g.s), out_bytes = static_cast<uint32_t>(rows_in) * row_bytes;
  auto offset_of = [&](int block, int u) {
    const int col = block * kColsOfBlock + lc * 8;
    const uint32_t at = static_cast<uint32_t>(u * 8 + lr) * row_bytes + 2u * static_cast<uint32_t>(col);
    return !RAGGED || col < g.s ? at : 0x80000000u;
  };

  // scores, rounded and packed in pairs of columns: of the lane's row, columns 64 block + 32 i + 8 q + 4 half + 0..3
  uint32_t sp[NBW][2][8];
  float mx = -INFINITY;
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int block = wave + WAVES * t;
    if (block >= active) break;
    const bool next = t + 1 < NBW && block + WAVES < active;
    floatx16_t acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
#pragma unroll
    for (int step = 0; step < kSteps; ++step) {
      if (t > 0 || step > 0) wait_vmcnt<0>();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int kk = 0; kk < KD / 16; ++kk) {
        const Frag<true> fa = SQ::fragment(sQ + (kk >> 2) * SQ::kElems, 0, kk & 3, lane);
#pragma unroll
        for (int j = 0; j < 2 / kSteps; ++j) {
          const Frag<true> fb = SK::fragment(sK + (kk >> 2) * SK::kElems, 32 * j, kk & 3, lane);
          const int i = step * (2 / kSteps) + j;
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb.operand(), fa.operand(), acc[i], 0, 0, 0);
        }
      }
      // this wavefront has read its K: the next rows may take its place (unless S is staged there first)
      wait_lgkmcnt0();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (step + 1 < kSteps) load_k(block * kColsOfBlock + (step + 1) * kStepCols);
      else if (next && g.S == nullptr) load_k((block + WAVES) * kColsOfBlock);
    }
    if (g.S != nullptr) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd)
          stage_write(i, qd, make_uint2(pack_bf16(acc[i][4 * qd], acc[i][4 * qd + 1]), pack_bf16(acc[i][4 * qd + 2], acc[i][4 * qd + 3])));
      const RowBuffer out = row_buffer(g.S + out0, out_bytes);
#pragma unroll
      for (int u = 0; u < 4; ++u) store_row(out, offset_of(block, u), stage_read(u), g.stream_s != 0);
      wait_lgkmcnt0();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (next) load_k((block + WAVES) * kColsOfBlock);
    }
    // columns beyond the diagonal, in its block only
    if (block == active - 1) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int col = block * kColsOfBlock + 32 * i + 8 * (r >> 2) + 4 * half + (r & 3);
          acc[i][r] = col <= my_row ? acc[i][r] : -INFINITY;
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        mx = fmaxf(fmaxf(acc[i][2 * r], acc[i][2 * r + 1]), mx);
        sp[t][i][r] = pack_bf16(acc[i][2 * r], acc[i][2 * r + 1]);
      }
  }
  // Row maximum.  Rounding to storage and the positive scale are monotonic, so the largest logit is that of the
  // largest score before rounding.
  mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
  if (lane < 32) row_max[wave * kRowsOfBlock + lane] = mx;
  block_barrier();
#pragma unroll
  for (int w = 0; w < WAVES; ++w) mx = fmaxf(mx, row_max[w * kRowsOfBlock + (lane & 31)]);
  const float m = softmax_logit(round_to_storage(mx, static_cast<bf16_t*>(nullptr)), g.scale);
  float e[kKeep ? NBW : 1][2][16];
  auto exponentials = [&](int t, float (&x)[2][16]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        x[i][2 * r] = softmax_exp(softmax_logit(bf16_lo(sp[t][i][r]), g.scale), m);
        x[i][2 * r + 1] = softmax_exp(softmax_logit(bf16_hi(sp[t][i][r]), g.scale), m);
      }
  };
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int block = wave + WAVES * t;
    if (block >= active) break;
    float (&x)[2][16] = e[kKeep ? t : 0];
    exponentials(t, x);
    float v[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int i = n >> 2, qd = n & 3;
      v[n] = softmax_group4(x[i][4 * qd], x[i][4 * qd + 1], x[i][4 * qd + 2], x[i][4 * qd + 3]);
    }
    const float th = softmax_tree8(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7]);
    const float sum = th + __shfl_xor(th, 32, kWave);
    if (lane < 32) block_sum[block * kRowsOfBlock + lane] = sum;
  }
  block_barrier();
  // blocks alternately into two running sums, one per half of the wavefront
  float sum = 0.f;
  for (int b = 0; b < active; b += 2) {
    const float x = block_sum[min(b + half, kMaxBlocks - 1) * kRowsOfBlock + (lane & 31)];
    sum += b + half < active ? x : 0.f;
  }
  const float inv = softmax_inverse(sum + __shfl_xor(sum, 32, kWave));

  const RowBuffer out_p = row_buffer(g.P + out0, g.P != nullptr ? out_bytes : 0u);
  const RowBuffer out_pd = row_buffer(g.Pd + out0, g.Pd != nullptr ? out_bytes : 0u);
  // dropout group (8 columns) of this lane in row lr, block 0
  const uint64_t group0 = ((((static_cast<uint64_t>(z1) * g.global_heads + g.head0 + z2) * g.s + r0 + lr) * static_cast<uint64_t>(g.s)) >> 3) + lc;
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int block = wave + WAVES * t;
    if (block >= active) break;
    if (!kKeep) exponentials(t, e[0]);
    const float (&x)[2][16] = e[kKeep ? t : 0];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        stage_write(i, qd, make_uint2(pack_bf16(x[i][4 * qd] * inv, x[i][4 * qd + 1] * inv),
                                      pack_bf16(x[i][4 * qd + 2] * inv, x[i][4 * qd + 3] * inv)));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uintx4_t raw = stage_read(u);
      const uint32_t at = offset_of(block, u);
      if (g.P != nullptr) store_row(out_p, at, raw, g.stream_p != 0);
      if (g.Pd != nullptr) {
        Raw8<bf16_t> r;
        r.v = make_uint4(raw[0], raw[1], raw[2], raw[3]);
        float p[8];
        unpack(r, p);
        dropout_apply8(g.key, group0 + static_cast<uint64_t>(u * g.s + block * (kColsOfBlock / 8)), p);
        row_buffer_store(out_pd, at, uintx4_t{pack_bf16(p[0], p[1]), pack_bf16(p[2], p[3]), pack_bf16(p[4], p[5]), pack_bf16(p[6], p[7])});
      }
    }
  }
  // zeros between the diagonal's block and the next multiple of 128 columns (at most one block)
  if (blocks > active && wave == (active & (WAVES - 1))) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uintx4_t zero = {0u, 0u, 0u, 0u};
      if (g.P != nullptr) store_row(out_p, offset_of(active, u), zero, g.stream_p != 0);
      if (g.Pd != nullptr) row_buffer_store(out_pd, offset_of(active, u), zero);
    }
  }
}

template <int KD, bool RAGGED, int WAVES, int NBW>
hipError_t launch(const ScoresSoftmaxArgs& g, hipStream_t st) {
  constexpr size_t smem = (kRowsOfBlock * KD + WAVES * kStepElems) * sizeof(bf16_t) + (WAVES + kMaxBlocks) * kRowsOfBlock * sizeof(float);
  auto kern = attn_scores_softmax_kernel<KD, RAGGED, WAVES, NBW>;
  LYNX_RAISE_LDS_LIMIT(kern, smem);
  hipLaunchKernelGGL(kern, dim3(g.row_blocks * g.nz), dim3(WAVES * kWave), smem, st, g);
  return hipGetLastError();
}
template <int KD, bool RAGGED>
hipError_t launch(const ScoresSoftmaxArgs& g, hipStream_t st) {
  // With so few workgroups that all run at once, one block per wavefront: the time of a workgroup is what counts.
  const bool few = static_cast<long long>(g.row_blocks) * g.nz <= 512;
  if (g.s <= 256 && few) return launch<KD, RAGGED, 4, 1>(g, st);
  if (g.s <= 512) return few ? launch<KD, RAGGED, 8, 1>(g, st) : launch<KD, RAGGED, 4, 2>(g, st);
  if (g.s <= 1024) return launch<KD, RAGGED, 8, 2>(g, st);
  return launch<KD, RAGGED, 8, 4>(g, st);
}

// ---- the gradient: dPd = dC V^T and the backward of dropout and softmax in one launch --------------------------------
// dS = scale P (dP - sum_j dP P), dP = keep c round(dPd), for s <= 1024.  The same split of rows and blocks: a wavefront forms
// its blocks of dPd, passes them through LDS into whole rows, where the dropout decisions are made, and keeps them,
// dropped elements cleared, beside the same elements of P (16 registers each per block of at most two) until the row
// sums are known.  dPd never goes through memory.  The sums are of the same terms as in softmax_dropout_bwd_kernel, which
// takes what is longer.  What bounds it: reading P and writing dS, then the vector ALU.  Two kernels and this one, us:
// 128 slices of 1024, d = 64, 112 and 83; 100 of 1000 101 and 72; 21 of 328, d = 104, 15 and 11; dQ and dK right behind it gain 5
// more, since dV then runs before it.  (The next block's V is asked for behind P, and only if there is one, so the compiler's
// waits for P count without it: most of V has landed before the arithmetic that it could hide behind.)
constexpr int kMaxGradientSeq = 1024;

struct ScoreGradientArgs {
  const bf16_t* dc; const bf16_t* v;
  const bf16_t* c;  // (row sums from C) row stride lddc
  long long lddc, ldv;
  const bf16_t* P; bf16_t* dS;
  int s, d, a, nz, row_blocks;
  int parts;  // (row sums from C) workgroups per 32 rows
  int global_heads, head0;
  float scale;
  DropoutKey key;
};

template <int KD, bool RAGGED, int WAVES, int NBW>
__global__ void __launch_bounds__(WAVES * kWave, WAVES == 8 ? 4 : 3) attn_score_gradient_kernel(ScoreGradientArgs g) {
  constexpr int kSlabs = KD / 64;
  constexpr int kStepCols = kStepElems / KD, kSteps = kColsOfBlock / kStepCols;
  using SQ = Slab<kRowsOfBlock, true, 64, 1>;
  using SK = Slab<kStepCols, true, 64, 1>;
  const int rb = g.row_blocks - 1 - static_cast<int>(blockIdx.x) / g.nz;
  const int bz = static_cast<int>(blockIdx.x) % g.nz;
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* sQ = reinterpret_cast<bf16_t*>(smem_raw);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  bf16_t* sK = sQ + kSlabs * SQ::kElems + wave * kStepElems;
  float* row_sum = reinterpret_cast<float*>(sQ + kSlabs * SQ::kElems + WAVES * kStepElems);  // [WAVES][32]
  const int z1 = bz / g.a, z2 = bz - z1 * g.a;
  const bf16_t* dc = g.dc + z1 * static_cast<long long>(g.s) * g.lddc + static_cast<long long>(z2) * g.d;
  const bf16_t* v = g.v + z1 * static_cast<long long>(g.s) * g.ldv + static_cast<long long>(z2) * g.d;
  const int r0 = rb * kRowsOfBlock;
  const int rows_in = RAGGED ? min(kRowsOfBlock, g.s - r0) : kRowsOfBlock;
  const int active = (r0 + rows_in - 1) / kColsOfBlock + 1;
  const int padded = min(g.s, (r0 + rows_in + 127) / 128 * 128);
  const int blocks = (padded + kColsOfBlock - 1) / kColsOfBlock;

  auto load_v = [&](int col) {
#pragma unroll
    for (int sl = 0; sl < kSlabs; ++sl) load_rows<SK, KD, RAGGED>(v, g.ldv, g.s, g.d, col, sl, sK + sl * SK::kElems, lane);
  };
  if (wave < kSlabs) load_rows<SQ, KD, RAGGED>(dc, g.lddc, g.s, g.d, r0, wave, sQ + wave * SQ::kElems, lane);
  if (wave < active) load_v(wave * kColsOfBlock);
  wait_vmcnt<0>();
  block_barrier();

  const int my_row = r0 + (lane & 31), half = lane >> 5;
  const int lr = lane >> 3, lc = lane & 7;
  // (staging as above)
  bf16_t* const stage_to = sK + (lane & 31) * kColsOfBlock + 4 * (half ^ ((lane >> 4) & 1));
  auto stage_read = [&](int u) {
    const int row = u * 8 + lr;
    const uintx4_t x = *reinterpret_cast<const uintx4_t*>(sK + row * kColsOfBlock + ((lc ^ ((row >> 1) & 7)) << 3));
    return u < 2 ? x : uintx4_t{x[2], x[3], x[0], x[1]};
  };
  const long long out0 = (static_cast<long long>(bz) * g.s + r0) * g.s;
  const uint32_t row_bytes = 2u * static_cast<uint32_t>(g.s), out_bytes = static_cast<uint32_t>(rows_in) * row_bytes;
  auto offset_of = [&](int block, int u) {
    const int col = block * kColsOfBlock + lc * 8;
    const uint32_t at = static_cast<uint32_t>(u * 8 + lr) * row_bytes + 2u * static_cast<uint32_t>(col);
    return !RAGGED || col < g.s ? at : 0x80000000u;
  };
  const RowBuffer in_p = row_buffer(g.P + out0, out_bytes), out = row_buffer(g.dS + out0, out_bytes);
  const uint64_t group0 = ((((static_cast<uint64_t>(z1) * g.global_heads + g.head0 + z2) * g.s + r0 + lr) * static_cast<uint64_t>(g.s)) >> 3) + lc;

  uintx4_t dpd[NBW][4], pr[NBW][4];  // dPd (dropped elements cleared) and P in rows
  float dot[4] = {0.f, 0.f, 0.f, 0.f};
  auto unpacked = [](uintx4_t raw, float (&x)[8]) {
    Raw8<bf16_t> r;
    r.v = make_uint4(raw[0], raw[1], raw[2], raw[3]);
    unpack(r, x);
  };
  // dP of eight elements: cleared ones stay zero
  auto gradient8 = [&](uintx4_t raw, float (&x)[8]) {
    unpacked(raw, x);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] *= g.key.scale;
  };
  DropoutKey keep_only = g.key;  // (1 or 0 of each element: the raw value, or cleared)
  keep_only.scale = 1.0f;
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int block = wave + WAVES * t;
    if (block >= active) break;
    const bool next = t + 1 < NBW && block + WAVES < active;
    floatx16_t acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
#pragma unroll
    for (int step = 0; step < kSteps; ++step) {
      if (t > 0 || step > 0) wait_vmcnt<0>();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int kk = 0; kk < KD / 16; ++kk) {
        const Frag<true> fa = SQ::fragment(sQ + (kk >> 2) * SQ::kElems, 0, kk & 3, lane);
#pragma unroll
        for (int j = 0; j < 2 / kSteps; ++j) {
          const Frag<true> fb = SK::fragment(sK + (kk >> 2) * SK::kElems, 32 * j, kk & 3, lane);
          const int i = step * (2 / kSteps) + j;
          acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb.operand(), fa.operand(), acc[i], 0, 0, 0);
        }
      }
      wait_lgkmcnt0();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (step + 1 < kSteps) load_v(block * kColsOfBlock + (step + 1) * kStepCols);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) pr[t][u] = row_buffer_load(in_p, offset_of(block, u));
    if (block == active - 1) {  // nothing beyond the diagonal
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int col = block * kColsOfBlock + 32 * i + 8 * (r >> 2) + 4 * half + (r & 3);
          acc[i][r] = col <= my_row ? acc[i][r] : 0.f;
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        *reinterpret_cast<uint2*>(stage_to + (((4 * i + qd) ^ ((lane >> 1) & 7)) << 3)) =
            make_uint2(pack_bf16(acc[i][4 * qd], acc[i][4 * qd + 1]), pack_bf16(acc[i][4 * qd + 2], acc[i][4 * qd + 3]));
#pragma unroll
    for (int u = 0; u < 4; ++u) dpd[t][u] = stage_read(u);
    wait_lgkmcnt0();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (next) load_v((block + WAVES) * kColsOfBlock);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float x[8], p[8];
      unpacked(dpd[t][u], x);
      dropout_apply8(keep_only, group0 + static_cast<uint64_t>(u * g.s + block * (kColsOfBlock / 8)), x);
      dpd[t][u] = uintx4_t{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7])};
      unpacked(pr[t][u], p);
#pragma unroll
      for (int i = 0; i < 8; ++i) dot[u] += (x[i] * g.key.scale) * p[i];
    }
  }
  // row sums: over a row's eight lanes, then over the wavefronts in order
#pragma unroll
  for (int u = 0; u < 4; ++u) dot[u] = group8_sum(dot[u]);
  if (lc == 0)
#pragma unroll
    for (int u = 0; u < 4; ++u) row_sum[wave * kRowsOfBlock + u * 8 + lr] = dot[u];
  block_barrier();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    dot[u] = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) dot[u] += row_sum[w * kRowsOfBlock + u * 8 + lr];
  }
#pragma unroll
  for (int t = 0; t < NBW; ++t) {
    const int block = wave + WAVES * t;
    if (block >= active) break;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      float x[8], p[8];
      gradient8(dpd[t][u], x);
      unpacked(pr[t][u], p);
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = softmax_bwd(p[i], x[i], dot[u], g.scale);
      row_buffer_store(out, offset_of(block, u), uintx4_t{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7])});
    }
  }
  if (blocks > active && wave == (active & (WAVES - 1))) {
#pragma unroll
    for (int u = 0; u < 4; ++u) row_buffer_store(out, offset_of(active, u), uintx4_t{0u, 0u, 0u, 0u});
  }
}

// Head dimension 128, whole tiles of 128 rows, the row sums known beforehand: as sum_dd dC[i, dd] C[i, dd], with the bits of
// attn_rowdot and attn_dscores_kernel.  A block is finished and stored as soon as it is multiplied.  (A kernel of its own: as a
// form of the one above it took that one's registers, 128 slices of 1024, d = 64, 86 -> 135 us.)  The buffer descriptors are more
// than the scalar registers hold: 60 and more of them are kept in lanes of vector registers, which the block loop reads back.
// The blocks of a row do not need each other, so `parts` workgroups divide them where there are few rows; each forms the sums of
// its rows.  (V asked for whether or not a block follows, so that the waits for P do not include it: no faster at any of 58
// sizes, and 1 to 1.8 % of a pass slower with 64 slices of 1024 or 128 of 512, for the loads after the last block.)
template <int WAVES>
__global__ void __launch_bounds__(WAVES * kWave, WAVES == 8 ? 4 : 3) attn_score_gradient_from_c_kernel(ScoreGradientArgs g) {
  constexpr int KD = 128, kSlabs = KD / 64, kStepCols = kStepElems / KD, kSteps = kColsOfBlock / kStepCols;
  using SQ = Slab<kRowsOfBlock, true, 64, 1>;
  using SK = Slab<kStepCols, true, 64, 1>;
  const int of_rows = g.nz * g.parts, rest = static_cast<int>(blockIdx.x) % of_rows;
  const int rb = g.row_blocks - 1 - static_cast<int>(blockIdx.x) / of_rows;
  const int part = rest / g.nz, bz = rest - part * g.nz;
  extern __shared__ __align__(1024) unsigned char smem_raw[];
  bf16_t* sQ = reinterpret_cast<bf16_t*>(smem_raw);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  bf16_t* sK = sQ + kSlabs * SQ::kElems + wave * kStepElems;
  float* row_sum = reinterpret_cast<float*>(sQ + kSlabs * SQ::kElems + WAVES * kStepElems);  // [32]
  const int z1 = bz / g.a, z2 = bz - z1 * g.a;
  const long long head = z1 * static_cast<long long>(g.s) * g.lddc + static_cast<long long>(z2) * KD;
  const bf16_t* dc = g.dc + head;
  const bf16_t* v = g.v + z1 * static_cast<long long>(g.s) * g.ldv + static_cast<long long>(z2) * KD;
  const int r0 = rb * kRowsOfBlock;
  const int active = (r0 + kRowsOfBlock - 1) / kColsOfBlock + 1;
  const int blocks = (r0 + kRowsOfBlock + 127) / 128 * 128 / kColsOfBlock;

  auto load_v = [&](int col) {
#pragma unroll
    for (int sl = 0; sl < kSlabs; ++sl) load_rows<SK, KD, false>(v, g.ldv, g.s, KD, col, sl, sK + sl * SK::kElems, lane);
  };
  if (wave < kSlabs) load_rows<SQ, KD, false>(dc, g.lddc, g.s, KD, r0, wave, sQ + wave * SQ::kElems, lane);
  const int first = part * WAVES + wave, step_blocks = g.parts * WAVES;
  if (first < active) load_v(first * kColsOfBlock);
#pragma unroll
  for (int i = 0; i < kRowsOfBlock / (4 * WAVES); ++i) {
    const int row = 4 * (wave + WAVES * i) + (lane >> 4);
    const long long at = (r0 + row) * g.lddc;
    const float dot = row_dot16(lane & 15, KD, [&](int v8, float (&x)[8]) { load8(dc + at + v8 * 8, x); },
                                [&](int v8, float (&x)[8]) { load8_streaming(g.c + head + at + v8 * 8, x); });
    if ((lane & 15) == 0) row_sum[row] = dot;
  }
  wait_vmcnt<0>();
  block_barrier();

  const int my_row = r0 + (lane & 31), half = lane >> 5;
  const int lr = lane >> 3, lc = lane & 7;
  // (staging as above)
  bf16_t* const stage_to = sK + (lane & 31) * kColsOfBlock + 4 * (half ^ ((lane >> 4) & 1));
  auto stage_read = [&](int u) {
    const int row = u * 8 + lr;
    const uintx4_t x = *reinterpret_cast<const uintx4_t*>(sK + row * kColsOfBlock + ((lc ^ ((row >> 1) & 7)) << 3));
    return u < 2 ? x : uintx4_t{x[2], x[3], x[0], x[1]};
  };
  const long long out0 = (static_cast<long long>(bz) * g.s + r0) * g.s;
  const uint32_t row_bytes = 2u * static_cast<uint32_t>(g.s), out_bytes = kRowsOfBlock * row_bytes;
  auto offset_of = [&](int block, int u) {
    return static_cast<uint32_t>(u * 8 + lr) * row_bytes + 2u * static_cast<uint32_t>(block * kColsOfBlock + lc * 8);
  };
  const RowBuffer in_p = row_buffer(g.P + out0, out_bytes), out = row_buffer(g.dS + out0, out_bytes);
  const uint64_t group0 = ((((static_cast<uint64_t>(z1) * g.global_heads + g.head0 + z2) * g.s + r0 + lr) * static_cast<uint64_t>(g.s)) >> 3) + lc;
  float dot[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) dot[u] = row_sum[u * 8 + lr];
#pragma unroll 1
  for (int block = first; block < active; block += step_blocks) {
    floatx16_t acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
#pragma unroll
    for (int step = 0; step < kSteps; ++step) {
      // (V was asked for ahead of the four stores of the block before; the waits for that block's P have seen to most of it)
      if (step > 0) wait_vmcnt<0>();
      else if (block != first) wait_vmcnt<4>();
      asm volatile("" ::: "memory");
#pragma unroll
      for (int kk = 0; kk < KD / 16; ++kk) {
        const Frag<true> fa = SQ::fragment(sQ + (kk >> 2) * SQ::kElems, 0, kk & 3, lane);
        const Frag<true> fb = SK::fragment(sK + (kk >> 2) * SK::kElems, 0, kk & 3, lane);
        acc[step] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb.operand(), fa.operand(), acc[step], 0, 0, 0);
      }
      wait_lgkmcnt0();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (step + 1 < kSteps) load_v(block * kColsOfBlock + (step + 1) * kStepCols);
    }
    uintx4_t pr[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) pr[u] = row_buffer_load(in_p, offset_of(block, u));
    if (block == active - 1) {  // nothing beyond the diagonal
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int col = block * kColsOfBlock + 32 * i + 8 * (r >> 2) + 4 * half + (r & 3);
          acc[i][r] = col <= my_row ? acc[i][r] : 0.f;
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        *reinterpret_cast<uint2*>(stage_to + (((4 * i + qd) ^ ((lane >> 1) & 7)) << 3)) =
            make_uint2(pack_bf16(acc[i][4 * qd], acc[i][4 * qd + 1]), pack_bf16(acc[i][4 * qd + 2], acc[i][4 * qd + 3]));
    uintx4_t rows[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) rows[u] = stage_read(u);
    wait_lgkmcnt0();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (block + step_blocks < active) load_v((block + step_blocks) * kColsOfBlock);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      Raw8<bf16_t> raw_x, raw_p;
      raw_x.v = make_uint4(rows[u][0], rows[u][1], rows[u][2], rows[u][3]);
      raw_p.v = make_uint4(pr[u][0], pr[u][1], pr[u][2], pr[u][3]);
      float x[8], p[8];
      unpack(raw_x, x);
      unpack(raw_p, p);
      dropout_apply8(g.key, group0 + static_cast<uint64_t>(u * g.s + block * (kColsOfBlock / 8)), x);
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = softmax_bwd(p[i], x[i], dot[u], g.scale);
      row_buffer_store(out, offset_of(block, u), uintx4_t{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3]), pack_bf16(x[4], x[5]), pack_bf16(x[6], x[7])});
    }
  }
  if (blocks > active && first == active % step_blocks) {
#pragma unroll
    for (int u = 0; u < 4; ++u) row_buffer_store(out, offset_of(active, u), uintx4_t{0u, 0u, 0u, 0u});
  }
}

template <int WAVES>
hipError_t launch_from_c(const ScoreGradientArgs& g, hipStream_t st) {
  constexpr size_t smem = (kRowsOfBlock * 128 + WAVES * kStepElems) * sizeof(bf16_t) + kRowsOfBlock * sizeof(float);
  auto kern = attn_score_gradient_from_c_kernel<WAVES>;
  LYNX_RAISE_LDS_LIMIT(kern, smem);
  hipLaunchKernelGGL(kern, dim3(g.row_blocks * g.nz * g.parts), dim3(WAVES * kWave), smem, st, g);
  return hipGetLastError();
}

template <int KD, bool RAGGED, int WAVES, int NBW>
hipError_t launch(const ScoreGradientArgs& g, hipStream_t st) {
  constexpr size_t smem = (kRowsOfBlock * KD + WAVES * kStepElems) * sizeof(bf16_t) + WAVES * kRowsOfBlock * sizeof(float);
  auto kern = attn_score_gradient_kernel<KD, RAGGED, WAVES, NBW>;
  LYNX_RAISE_LDS_LIMIT(kern, smem);
  hipLaunchKernelGGL(kern, dim3(g.row_blocks * g.nz), dim3(WAVES * kWave), smem, st, g);
  return hipGetLastError();
}
template <int KD, bool RAGGED>
hipError_t launch(const ScoreGradientArgs& g, hipStream_t st) {
  const bool few = static_cast<long long>(g.row_blocks) * g.nz <= 512;
  if (g.s <= 256 && few) return launch<KD, RAGGED, 4, 1>(g, st);
  if (g.s <= 512) return few ? launch<KD, RAGGED, 8, 1>(g, st) : launch<KD, RAGGED, 4, 2>(g, st);
  return launch<KD, RAGGED, 8, 2>(g, st);
}

}  // namespace

// (32 rows per workgroup: with 2^23 of them and more the kernels of 128 rows may still be launched)
bool attn_scores_softmax_supported(int dtype, int s, int d, long long ld, long long slices) {
  return dtype == 1 && s % 8 == 0 && s <= kMaxSeq && d % 8 == 0 && d <= 128 && ld % 8 == 0 && ld < (1ll << 28) &&
         fits_grid((s + kRowsOfBlock - 1) / kRowsOfBlock * slices, 8 * kWave);
}

hipError_t attn_scores_softmax_fwd(const void* q, const void* k, long long ld, void* S, void* P, void* Pd, AttnShape sh, int d,
                                   float scale, DropoutParams dp, hipStream_t st) {
  if (!attn_scores_softmax_supported(1, sh.s, d, ld, static_cast<long long>(sh.a) * sh.b)) return hipErrorInvalidValue;
  ScoresSoftmaxArgs g{};
  g.q = static_cast<const bf16_t*>(q); g.k = static_cast<const bf16_t*>(k); g.ld = ld;
  g.S = static_cast<bf16_t*>(S); g.P = static_cast<bf16_t*>(P); g.Pd = static_cast<bf16_t*>(Pd);
  g.s = sh.s; g.d = d; g.a = sh.a; g.nz = sh.a * sh.b;
  g.row_blocks = (sh.s + kRowsOfBlock - 1) / kRowsOfBlock;
  g.global_heads = sh.global_heads; g.head0 = sh.head0;
  g.scale = scale;
  g.key = make_dropout_key(dp, 0);
  // as in the kernels that this one replaces: S is not read again soon, nor is P where Pd is written too; rows that end
  // inside a 128-byte line are left to the caches
  const bool whole_lines = sh.s % 64 == 0;
  g.stream_s = whole_lines;
  g.stream_p = whole_lines && Pd != nullptr;
  const bool whole = sh.s % kColsOfBlock == 0 && (d == 64 || d == 128);
  if (d <= 64) return whole ? launch<64, false>(g, st) : launch<64, true>(g, st);
  return whole ? launch<128, false>(g, st) : launch<128, true>(g, st);
}

bool attn_score_gradient_supported(int dtype, int s, int d, long long ld, long long slices) {
  return s <= kMaxGradientSeq && attn_scores_softmax_supported(dtype, s, d, ld, slices);
}

// Workgroups of eight wavefronts that share 32 rows of attn_score_gradient_from_c_kernel.
static long long attn_score_gradient_parts(int s, long long slices) {
  const long long blocks = (s + kColsOfBlock - 1) / kColsOfBlock, most = (blocks + 7) / 8;
  const long long at_once = 512 / ((s + kRowsOfBlock - 1) / kRowsOfBlock * slices);  // two per compute unit
  return at_once < 1 ? 1 : at_once < most ? at_once : most;
}

// Head dimension 128 and whole tiles of 128 rows, where attn_rowdot and attn_dscores_kernel are the alternative, up to
// 2^26 elements of dS and 3072 groups of 32 rows.  Those two walk tiles of 128 rows and so read V a quarter as often, which is what
// counts once P and dS, 256 MB together, outgrow the memory-side cache, or with many short rows; this one is a launch less
// and has four times the workgroups.  Passes with those two and with this one, us: 4 slices of s = 512 100 and 96, 64 of 768 282 and
// 277, 256 of 384 382 and 382, 192 of 512 410 and 410, 64 of 1024 369 and 362; beyond: 448 of 384 582 and 596, 512 of 256 432 and
// 439, 256 of 512 495 and 500, 1024 of 128 401 and 404.  The kernels with the launch of dQ and dK behind them beyond 2^26:
// 128 of 1024 189 and 198, 40 of 2048 194 and 198, 64 of 2048 310 and 329.  Few long rows, whose workgroups share them:
// one slice of 2048 148 and 145 (with a workgroup per 32 rows 154), three 162 and 160 (165), one of 1536 137 and 134 (140).
bool attn_score_gradient_from_c(int dtype, int s, int d, long long ld, long long slices) {
  return d == 128 && s % 128 == 0 && s <= kMaxSeq && slices * s * s <= (1ll << 26) && s / kRowsOfBlock * slices <= 3072 &&
         attn_scores_softmax_supported(dtype, s, d, ld, slices);
}

hipError_t attn_score_gradient(const void* dc, long long lddc, const void* v, long long ldv, const void* c, const void* P, void* dS,
                               AttnShape sh, int d, float scale, DropoutParams dp, hipStream_t st) {
  const long long slices = static_cast<long long>(sh.a) * sh.b;
  const bool from_c = c != nullptr;
  if (lddc > ldv || !(from_c ? attn_score_gradient_from_c(1, sh.s, d, ldv, slices) : attn_score_gradient_supported(1, sh.s, d, ldv, slices)))
    return hipErrorInvalidValue;
  ScoreGradientArgs g{};
  g.dc = static_cast<const bf16_t*>(dc); g.lddc = lddc;
  g.v = static_cast<const bf16_t*>(v); g.ldv = ldv;
  g.c = static_cast<const bf16_t*>(c);
  g.P = static_cast<const bf16_t*>(P); g.dS = static_cast<bf16_t*>(dS);
  g.s = sh.s; g.d = d; g.a = sh.a; g.nz = sh.a * sh.b;
  g.row_blocks = (sh.s + kRowsOfBlock - 1) / kRowsOfBlock;
  g.global_heads = sh.global_heads; g.head0 = sh.head0;
  g.scale = scale;
  g.key = make_dropout_key(dp, 0);
  if (from_c) {
    g.parts = 1;
    if (sh.s <= 256 && static_cast<long long>(g.row_blocks) * g.nz <= 512) return launch_from_c<4>(g, st);
    // as many as leave the longest row one block per wavefront, if they run at once
    g.parts = static_cast<int>(attn_score_gradient_parts(sh.s, slices));
    return launch_from_c<8>(g, st);
  }
  const bool whole = sh.s % kColsOfBlock == 0 && (d == 64 || d == 128);
  if (d <= 64) return whole ? launch<64, false>(g, st) : launch<64, true>(g, st);
  return whole ? launch<128, false>(g, st) : launch<128, true>(g, st);
}

}  // namespace lynx
