// First stage of a plain column sum as a guest in another kernel's launch (the QKV bias gradient in that of the QKV
// weight and input gradients, which read the same tensor).  Its workgroups come between those of the longer contraction
// and the many short ones, and load ordinarily, so that the products behind them find the tensor in the caches.  Last in
// the launch and with streaming loads, they are what it waits for: passes of 432 tokens of h 640 in fp32 255.7 us without a guest,
// 259.1 with it last, 256.3 between; 192 of h 1024 260.5, 263.8, 259.7; 512 of h 576 261.9, 261.2, 260.7; in bf16 176 of h 3200
// 207.9, 209.8, 205.5; 80 of h 888 117.6, 118.7, 116.7; small layers 1 to 1.6 % less than without either way.
#pragma once
#include "device_common.h"
#include "kernels.h"

namespace lynx {

constexpr int kPartialRows = 32;  // rows of one partial, as in rows_colsum_kernel

struct ColumnPartials {
  const void* x;  // [rows, cols]
  float* part;    // [ceil(rows / 32), cols]
  int rows, cols;
  int tiles;      // of 32 rows x 64 vectors, one per wavefront
  int first, end; // workgroups, a multiple of 8 of them, so that those behind stay on their XCDs
};
// The guest of a launch of n workgroups of so many wavefronts, behind the first `first` of them.  Behind all of them where they
// have a unit each and the guest would push some onto a unit that has one: 400, 432 and 512 tokens of h 512 in fp32, 248 to 256
// workgroups, a pass without a guest 195.5, 198.9 and 211.5 us, with it between 199.7, 202.4 and 215.2, last 194.4, 196.7 and 208.9.
inline ColumnPartials guest_partials(const ColumnSumInput& in, int first, int n, int waves) {
  ColumnPartials c{};
  c.x = in.x; c.part = in.part;
  c.rows = in.rows; c.cols = in.cols;
  c.tiles = (in.rows + kPartialRows - 1) / kPartialRows * ((in.cols / 8 + kWave - 1) / kWave);
  const int groups = ((c.tiles + waves - 1) / waves + 7) / 8 * 8;
  c.first = n <= 256 && n + groups > 256 ? n : first;
  c.end = c.first + groups;
  return c;
}

// Tile `tile`, one vector of 8 columns per lane.  A lane has all 32 rows of its columns, so nothing goes through LDS,
// which belongs to the products; the order of the sums is that of rows_colsum_kernel: rows r, r + 4, ... of the tile
// form one sum, of four.
template <typename T>
__device__ __forceinline__ void column_partials(const ColumnPartials& c, int tile) {
  if (tile >= c.tiles) return;
  const int vecs = c.cols >> 3, wide = (vecs + kWave - 1) / kWave;
  const int block = tile / wide, vec = (tile - block * wide) * kWave + static_cast<int>(threadIdx.x & (kWave - 1));
  if (vec >= vecs) return;
  const int r0 = block * kPartialRows;
  const T* x = static_cast<const T*>(c.x) + static_cast<size_t>(r0) * c.cols + static_cast<size_t>(vec) * 8;
  float sum[4][8] = {};
  // 64 registers of rows.  A kernel with this guest takes 128 (bf16) and 140 (fp32) where the products alone take 66 and 100;
  // the ring in LDS leaves room for two and three of their workgroups per compute unit, which may have 256 and 168.
  constexpr int kAtOnce = sizeof(T) == 2 ? 16 : 8;
#pragma unroll
  for (int h = 0; h < kPartialRows; h += kAtOnce) {
    Raw8<T> raw[kAtOnce];
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k)
      if (r0 + h + k < c.rows) load_raw(x + static_cast<size_t>(h + k) * c.cols, raw[k]);
#pragma unroll
    for (int k = 0; k < kAtOnce; ++k) {
      if (r0 + h + k >= c.rows) break;
      float v[8];
      unpack(raw[k], v);
#pragma unroll
      for (int i = 0; i < 8; ++i) sum[k & 3][i] += v[i];
    }
  }
  float total[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) total[i] = (sum[0][i] + sum[1][i]) + (sum[2][i] + sum[3][i]);
  store8(c.part + static_cast<size_t>(block) * c.cols + static_cast<size_t>(vec) * 8, total);
}

}  // namespace lynx
