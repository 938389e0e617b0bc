// Building blocks of the matrix-core kernels: MFMA operand fragments, the LDS slab layouts
// that direct global -> LDS loads fill and fragment reads drain without bank conflicts, and
// the hand-counted waits those loads need.  Shared by the dense products (gemm_mfma.hip) and
// the fused attention kernels (attn_fused.hip); everything here is device code in an
// anonymous namespace of the including file.
#pragma once
#include "device_common.h"

namespace lynx {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short short4_t __attribute__((ext_vector_type(4)));
typedef unsigned int uintx4_t __attribute__((ext_vector_type(4)));
typedef unsigned int uintx2_t __attribute__((ext_vector_type(2)));
typedef short short8_t __attribute__((ext_vector_type(8)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));

constexpr int kBK = 32;        // K slab
constexpr int kThreads = 256;  // 4 wavefronts
constexpr int kWaves = kThreads / kWave;

// s_waitcnt with only the vector-memory counter constrained (gfx9 encoding:
// vmcnt = bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
__device__ __forceinline__ void wait_lgkmcnt0() {
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (0 << 8));
}
// Waits until at most n newer slabs of LOADS loads each are still in flight (n is uniform).
template <int LOADS, int MOST>
__device__ __forceinline__ void wait_slabs(int n) {
  if constexpr (MOST == 0) wait_vmcnt<0>();
  else if (n >= MOST) wait_vmcnt<MOST * LOADS>();
  else wait_slabs<LOADS, MOST - 1>(n);
}

// Workgroup barrier that neither the optimiser nor the scheduler moves memory
// accesses across (and that, unlike __syncthreads, does not drain the loads
// still in flight).  This wavefront's LDS accesses are complete before it: a
// fragment that is merely requested when the barrier opens can be overtaken by
// another wavefront's writes to the buffer the barrier releases.  (WAITED: the
// caller has just waited for them.)
template <bool WAITED = false>
__device__ __forceinline__ void block_barrier() {
  asm volatile("" ::: "memory");
  if (!WAITED) wait_lgkmcnt0();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef const __attribute__((address_space(1))) void* global_void_ptr;

// Direct load of 16 bytes per lane from `base` (uniform) + offset to LDS at `to` (uniform) + 16 lane: a raw buffer that
// starts at `base`, with no bound but that of the 32-bit offsets.
__device__ __forceinline__ void buffer_load_to_lds(const void* base, uint32_t offset, bf16_t* to) {
#if defined(__HIP_DEVICE_COMPILE__)  // (the host pass does not know the resource type)
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0xFFFFFFFF, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)(to), 16, offset, 0, 0, 0);
#endif
}

// `bytes` bytes from `base` (both uniform) as a raw buffer: 16-byte accesses at 32-bit offsets, of which those at or
// beyond `bytes` read zeros and write nothing.
struct RowBuffer {
#if defined(__HIP_DEVICE_COMPILE__)
  __amdgpu_buffer_rsrc_t rsrc;
#endif
};
__device__ __forceinline__ RowBuffer row_buffer(const void* base, uint32_t bytes) {
  RowBuffer b;
#if defined(__HIP_DEVICE_COMPILE__)
  b.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
#endif
  return b;
}
__device__ __forceinline__ uintx4_t row_buffer_load(const RowBuffer& b, uint32_t offset) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_raw_buffer_load_b128(b.rsrc, offset, 0, 0);
#else
  return uintx4_t{};
#endif
}
__device__ __forceinline__ void row_buffer_store(const RowBuffer& b, uint32_t offset, uintx4_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_buffer_store_b128(v, b.rsrc, offset, 0, 0);
#endif
}
// ... with the non-temporal hint
__device__ __forceinline__ void row_buffer_store_streaming(const RowBuffer& b, uint32_t offset, uintx4_t v) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_raw_buffer_store_b128(v, b.rsrc, offset, 0, 2);
#endif
}

// An MFMA operand fragment as it arrives from LDS.  K-major slabs are read with plain
// 16-byte loads, which the compiler tracks.  MN-major slabs are read with the transposing
// LDS read, issued as inline assembly: the compiler's hazard tracking takes that read, as
// a builtin, to alias every direct-to-LDS load in flight and waits for all of them
// (vmcnt(0)) before it, which empties the prefetch ring once per slab.  The kernel's own
// lgkmcnt waits cover these reads; settle(), called after such a wait, makes every later
// use of the registers depend on a point after it.
template <bool KMAJOR> struct Frag;
template <> struct Frag<true> {
  bf16x8_t v;
  __device__ __forceinline__ bf16x8_t operand() const { return v; }
  __device__ __forceinline__ void settle() {}
};
template <> struct Frag<false> {
  short4_t lo, hi;
  __device__ __forceinline__ bf16x8_t operand() const {
    const short8_t v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8_t, v);
  }
  __device__ __forceinline__ void settle() { asm volatile("" : "+v"(lo), "+v"(hi)); }
};

// One slab (ROWS x BK elements) of an operand, BK = 32 or 64, loaded by WAVES wavefronts.
template <int ROWS, bool KMAJOR, int BK = kBK, int WAVES = kWaves>
struct Slab {
  static constexpr int kElems = ROWS * BK;
  static constexpr int kLoadsPerWave = kElems / 512 / WAVES;  // 1 KB direct loads per wavefront
  static constexpr int kLanesPerRow = BK / 8;               // K-major: 16-byte chunks per row
  static constexpr int kRowChunks = ROWS / 8;               // MN-major: 16-byte chunks per k-row
  static constexpr int kRowsPerLoad = 64 / kRowChunks;      // MN-major: k-rows per 1 KB
  static_assert(kElems % (512 * WAVES) == 0 && (BK == 32 || BK == 64), "slab must split over the wavefronts");
  // 16-byte chunk permutation of row `row` of a K-major slab: 16 lanes of a fragment read are 16
  // consecutive rows, and their chunks have to fall into 16 different 16-byte columns of the 64
  // banks, of which a row covers a quarter (BK = 32) or half
  __device__ static __forceinline__ int kswz(int row) { return BK == 32 ? (row >> 2) & 3 : (row >> 1) & 7; }
  // ... and of k-row `k` of an MN-major slab: four consecutive k-rows in four different 64-byte
  // windows of the 64 banks (a row of 64 elements is half the banks wide, so its parity does half of it)
  __device__ static __forceinline__ int mnswz(int k) { return ROWS >= 128 ? (k & 3) << 2 : ((k >> 1) & 1) << 2; }

  // Which elements lane `lane` fetches in this wavefront's j-th load: 8 consecutive ones along
  // the contiguous index, starting at row mn and contraction index k of the slab.
  __device__ static __forceinline__ int lane_mn(int wave, int j, int lane) {
    const int q = wave + WAVES * j;  // which 1 KB piece of the slab
    if (KMAJOR) return (64 / kLanesPerRow) * q + lane / kLanesPerRow;
    return ((lane % kRowChunks) ^ mnswz(lane_k(wave, j, lane))) * 8;
  }
  __device__ static __forceinline__ int lane_k(int wave, int j, int lane) {
    const int q = wave + WAVES * j;
    if (KMAJOR) return ((lane % kLanesPerRow) ^ kswz(lane_mn(wave, j, lane))) * 8;
    return kRowsPerLoad * q + lane / kRowChunks;
  }
  // Global element offset of that fetch relative to the slab origin (row0, k0), and the
  // load's LDS offset.
  __device__ static __forceinline__ long long global_offset(int wave, int j, int lane, long long ld) {
    const long long mn = lane_mn(wave, j, lane), k = lane_k(wave, j, lane);
    return KMAJOR ? mn * ld + k : k * ld + mn;
  }
  __device__ static __forceinline__ int lds_offset(int wave, int j) { return (wave + WAVES * j) * 512; }

  // MFMA operand fragment of step ks: 8 consecutive k (at 16 ks + 8 (lane / 32)) of slab
  // row tile_row0 + lane % 32.
  __device__ static __forceinline__ Frag<KMAJOR> fragment(const bf16_t* slab, int tile_row0, int ks, int lane) {
    Frag<KMAJOR> f;
    if constexpr (KMAJOR) {
      const int r = tile_row0 + (lane & 31);
      const int chunk = (2 * ks + (lane >> 5)) ^ kswz(r);
      f.v = *reinterpret_cast<const bf16x8_t*>(slab + r * BK + chunk * 8);
    } else {
      // four blocks of 16 lanes: block b holds rows (b & 1) * 16.. of k-group b >> 1; in a
      // block, lane i points at k-row i / 4, columns 4 (i % 4)..+3 and receives column i.
      const int b = lane >> 4, i = lane & 15;
      const int k = ks * 16 + (b >> 1) * 8 + (i >> 2);
      const int col = tile_row0 + (b & 1) * 16 + ((i & 3) << 2);
      const int sw = mnswz(k);  // same for k and k + 4
      const bf16_t* p = slab + k * ROWS + (((col >> 3) ^ sw) << 3) + (col & 7);
      typedef const __attribute__((address_space(3))) bf16_t* lds_ptr_t;
      const uint32_t addr = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_ptr_t)(p)));
      asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(f.lo) : "v"(addr));
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.hi) : "v"(addr), "n"(4 * ROWS * 2));
    }
    return f;
  }
};

}  // namespace
}  // namespace lynx
