// HBM-bound elementwise kernels: GeLU forward/backward, bias+dropout+residual,
// dropout backward, column sums (bias gradients) and the dropout-mask dump.
// Every thread moves 16-byte vectors of 8 elements; consecutive lanes touch
// consecutive vectors.  Column sums are two fixed-order stages (per row-block
// partials, then a serial sum over row-blocks), so results are deterministic.
#include "dropout_host.h"
#include "pointwise_math.h"
#include "device_common.h"

namespace lynx {
namespace {

constexpr int kThreads = 256;
constexpr int kRowsPerBlock = 32;  // rows folded into one column-sum partial

template <typename T>
__global__ void __launch_bounds__(kThreads) gelu_fwd_kernel(const T* __restrict__ u,
                                                            T* __restrict__ g, size_t nvec) {
  const size_t v = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (v >= nvec) return;
  float x[8];
  load8_streaming(u + v * 8, x);
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = gelu_f(x[i]);
  store8(g + v * 8, x);
}

// ---- per-element functors used with the column-sum frame ------------------
// apply(a, b, group, out): a, b = 8 elements of the one or two inputs, group =
// flat element index / 8; out = the 8 results, already rounded to storage.
template <typename T>
struct GeluBwdOp {  // du = dg * gelu'(u)
  static constexpr int kInputs = 2;
  static constexpr bool kStores = true;
  __device__ __forceinline__ void apply(const float (&a)[8], const float (&b)[8], size_t,
                                        float (&out)[8]) const {
    gelu_bwd8<T>(a, b, out);
  }
};

template <typename T>
struct DropoutBwdOp {  // din = keep * dout / (1 - p)
  static constexpr int kInputs = 1;
  static constexpr bool kStores = true;
  DropoutKey key;
  __device__ __forceinline__ void apply(const float (&a)[8], const float (&)[8], size_t group,
                                        float (&out)[8]) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = a[i];
    dropout_apply8(key, group, out);
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = round_to_storage(out[i], static_cast<T*>(nullptr));
  }
};

template <typename T>
struct IdentityOp {
  static constexpr int kInputs = 1;
  static constexpr bool kStores = false;
  __device__ __forceinline__ void apply(const float (&a)[8], const float (&)[8], size_t,
                                        float (&out)[8]) const {
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = a[i];
  }
};

// Frame: a workgroup owns a tile of kRowsPerBlock rows x 64 vectors (512 columns):
// wavefront w takes rows w, w + 4, ... of the tile, lane l the l-th vector, so every
// wavefront access is 1 KB contiguous and a thread's column stays fixed.  All of a
// thread's loads are issued before its first store; the four wavefronts' column sums
// are added in a fixed order through LDS.  Many small workgroups keep enough
// wavefronts resident to overlap the Philox / GeLU arithmetic with the memory traffic.
// V: vectors of the tile's width, 64 as above, or 16 where that gives the chip too few workgroups: then 16 lanes
// share a row, a thread has two rows instead of eight and four times the workgroups share the latency.
// The partial rows, their order of sums and with it their bits are the same: the narrow tile brings its 32 rows
// together in LDS, one column per thread (sums of the thread's two rows and then of the 16 row groups in series are
// another order, with 1.1 to 1.2 times the error against 64 bits in fp32).  Dropout backward, 64 -> 16 vectors:
// 256 x 256 fp32 6.6 -> 3.6 us, 768 x 512 bf16 6.8 -> 4.2, 984 x 3016 7.6 -> 6.0, 4000 x 1600 (500 workgroups of 64)
// 11.1 -> 8.4.
template <typename T, typename Op, int V>
__global__ void __launch_bounds__(kThreads)
rows_colsum_kernel(Op op, const T* in0, const T* __restrict__ in1, T* outp,  // outp may be in0
                   int rows, int cols, float* __restrict__ partial) {
  constexpr int kGroups = kThreads / V, kRowsPerThread = kRowsPerBlock / kGroups;
  constexpr bool kNarrow = V < kWave;
  constexpr int kSumRows = kThreads / kWave;  // rows r, r + 4, ... of the tile form one sum, of four
  __shared__ __align__(16) float sm[kNarrow ? kRowsPerBlock : kGroups][V][8];
  const int lane = threadIdx.x % V, w = threadIdx.x / V;
  const int vec = blockIdx.x * V + lane;
  const bool active = vec < (cols >> 3);
  const int r0 = blockIdx.y * kRowsPerBlock + w;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (active) {
    Raw8<T> ra[kRowsPerThread], rb[Op::kInputs == 2 ? kRowsPerThread : 1];
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
      const int r = r0 + k * kGroups;
      if (r < rows) {
        const size_t off = static_cast<size_t>(r) * cols + static_cast<size_t>(vec) * 8;
        load_raw_streaming(in0 + off, ra[k]);
        if (Op::kInputs == 2) load_raw_streaming(in1 + off, rb[Op::kInputs == 2 ? k : 0]);
      }
    }
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
      const int r = r0 + k * kGroups;
      float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (r < rows) {
        const size_t off = static_cast<size_t>(r) * cols + static_cast<size_t>(vec) * 8;
        float a[8], b[8] = {};
        unpack(ra[k], a);
        if (Op::kInputs == 2) unpack(rb[Op::kInputs == 2 ? k : 0], b);
        op.apply(a, b, off >> 3, v);
        if (Op::kStores) store8(outp + off, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += v[i];
      }
      if (kNarrow) store8(&sm[kNarrow ? w + k * kGroups : 0][lane][0], v);
    }
  }
  if (!kNarrow) store8(&sm[kNarrow ? 0 : w][lane][0], acc);
  __syncthreads();
  if (kNarrow) {  // one column per thread
    const int c = blockIdx.x * V * 8 + threadIdx.x;
    if (threadIdx.x < V * 8 && c < cols) {
      float t[kSumRows] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < kRowsPerBlock; ++r) t[r % kSumRows] += sm[kNarrow ? r : 0][threadIdx.x >> 3][threadIdx.x & 7];
      partial[static_cast<size_t>(blockIdx.y) * cols + c] = (t[0] + t[1]) + (t[2] + t[3]);
    }
  } else if (w == 0 && active) {
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = (sm[0][lane][i] + sm[1][lane][i]) + (sm[2][lane][i] + sm[3][lane][i]);
    store8(partial + static_cast<size_t>(blockIdx.y) * cols + static_cast<size_t>(vec) * 8, acc);
  }
}

// Workgroups of 64 vectors, two per compute unit: narrower tiles gain up to there (500: 11.1 -> 8.4 us; the plain
// sum, which is shorter, is level from 150 on: 4.6 us).  Larger grids keep whole-KB rows per wavefront access.
constexpr int kNarrowBelow = 512;

template <typename T, typename Op>
hipError_t launch_rows_colsum(Op op, const T* in0, const T* in1, T* outp, T* dbias, float* scratch,
                              int rows, int cols, ColumnSums* sums, hipStream_t st) {
  const int nvec = cols / 8;
  const int nrb = (rows + kRowsPerBlock - 1) / kRowsPerBlock;
  if ((nvec + kWave - 1) / kWave * nrb < kNarrowBelow)
    hipLaunchKernelGGL((rows_colsum_kernel<T, Op, 16>), dim3((nvec + 15) / 16, nrb), dim3(kThreads), 0, st, op, in0,
                       in1, outp, rows, cols, scratch);
  else
    hipLaunchKernelGGL((rows_colsum_kernel<T, Op, kWave>), dim3((nvec + kWave - 1) / kWave, nrb), dim3(kThreads), 0,
                       st, op, in0, in1, outp, rows, cols, scratch);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? sums->add(scratch, dbias, nrb, cols) : e;
}

// The second stage of every column sum of a backward pass in one launch (ColumnSums): a launch of
// one job takes 3 to 5 us, of which the reading is a fraction, and a backward had six.  All eight jobs:
// 256 tokens to 768 tokens of h 256 to 512: six launches 20 us -> 4; 16384 tokens of h 5120 (50 MB): 29 -> 14.
// Workgroup = 64 columns of one job x 16 row groups; group g adds partial rows g, g + 16, ... and the 16
// group sums are then added in order.
constexpr int kSumGroups = 16;
struct ColumnSumJobs {
  ColumnSums::Job job[ColumnSums::kMaxJobs];
  int end[ColumnSums::kMaxJobs];  // workgroups of jobs 0..i
};

template <typename T>
__global__ void __launch_bounds__(kSumGroups * kWave) column_sums_kernel(ColumnSumJobs jobs) {
  __shared__ float sm[kSumGroups][kWave];
  int block = static_cast<int>(blockIdx.x);
  ColumnSums::Job job = jobs.job[0];
  int first = 0;
#pragma unroll
  for (int i = 1; i < ColumnSums::kMaxJobs; ++i)
    if (block >= jobs.end[i - 1] && jobs.end[i] > 0) { job = jobs.job[i]; first = jobs.end[i - 1]; }
  block -= first;
  const int lane = threadIdx.x & (kWave - 1), grp = threadIdx.x / kWave;
  const int c = block * kWave + lane;
  float s = 0.f;
  if (c < job.cols) {
#pragma unroll 8
    for (int r = grp; r < job.rows; r += kSumGroups) s += job.part[static_cast<size_t>(r) * job.cols + c];
  }
  sm[grp][lane] = s;
  __syncthreads();
  if (grp == 0 && c < job.cols) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < kSumGroups; ++i) t += sm[i][lane];
    store1(static_cast<T*>(job.out) + c, t);
  }
}

template <typename T>
__global__ void __launch_bounds__(kThreads)
bias_dropout_add_kernel(const T* __restrict__ in, const T* __restrict__ bias,
                        const T* __restrict__ res, T* __restrict__ out, size_t nvec, int cols,
                        DropoutKey key) {
  const size_t v = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (v >= nvec) return;
  const size_t off = v * 8;
  const int c = static_cast<int>(off % static_cast<size_t>(cols));
  float a[8], b[8], r[8];
  load8(in + off, a);
  load8(bias + c, b);
  load8(res + off, r);
  float o[8];
  bias_dropout_add8(a, b, r, key, v, o);
  store8(out + off, o);
}

__global__ void __launch_bounds__(kThreads)
mask_bytes_kernel(uint8_t* __restrict__ out, size_t ngroups, uint64_t group0, DropoutKey key) {
  const size_t g = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x;
  if (g >= ngroups) return;
  const uint32_t keep = dropout_keep8(key, group0 + g);
  uint2 w;
  w.x = (keep & 1u) | ((keep & 2u) << 7) | ((keep & 4u) << 14) | ((keep & 8u) << 21);
  const uint32_t k2 = keep >> 4;
  w.y = (k2 & 1u) | ((k2 & 2u) << 7) | ((k2 & 4u) << 14) | ((k2 & 8u) << 21);
  *reinterpret_cast<uint2*>(out + g * 8) = w;
}

}  // namespace

hipError_t finish_column_sums(int dtype, ColumnSums* sums, hipStream_t st) {
  if (sums->n == 0) return hipSuccess;
  ColumnSumJobs jobs{};
  for (int i = 0; i < sums->n; ++i) {
    jobs.job[i] = sums->job[i];
    jobs.end[i] = (i > 0 ? jobs.end[i - 1] : 0) + (sums->job[i].cols + kWave - 1) / kWave;
  }
  const dim3 grid(jobs.end[sums->n - 1]), block(kSumGroups * kWave);
  sums->n = 0;
  if (dtype == 1) hipLaunchKernelGGL((column_sums_kernel<bf16_t>), grid, block, 0, st, jobs);
  else hipLaunchKernelGGL((column_sums_kernel<float>), grid, block, 0, st, jobs);
  return hipGetLastError();
}

size_t colsum_scratch_bytes(int rows, int cols) {
  const size_t nrb = (static_cast<size_t>(rows) + kRowsPerBlock - 1) / kRowsPerBlock;
  return nrb * static_cast<size_t>(cols) * sizeof(float);
}

hipError_t gelu_fwd(int dtype, const void* u, void* g, size_t n, hipStream_t st) {
  const size_t nvec = n / 8;
  const dim3 grid(static_cast<unsigned>((nvec + kThreads - 1) / kThreads));
  if (dtype == 1)
    hipLaunchKernelGGL((gelu_fwd_kernel<bf16_t>), grid, dim3(kThreads), 0, st,
                       static_cast<const bf16_t*>(u), static_cast<bf16_t*>(g), nvec);
  else
    hipLaunchKernelGGL((gelu_fwd_kernel<float>), grid, dim3(kThreads), 0, st,
                       static_cast<const float*>(u), static_cast<float*>(g), nvec);
  return hipGetLastError();
}

hipError_t gelu_bwd(int dtype, const void* dg, const void* u, void* du, void* dbias, float* scratch,
                    int rows, int cols, ColumnSums* sums, hipStream_t st) {
  if (dtype == 1) {
    return launch_rows_colsum(GeluBwdOp<bf16_t>{}, static_cast<const bf16_t*>(dg),
                              static_cast<const bf16_t*>(u), static_cast<bf16_t*>(du),
                              static_cast<bf16_t*>(dbias), scratch, rows, cols, sums, st);
  }
  return launch_rows_colsum(GeluBwdOp<float>{}, static_cast<const float*>(dg),
                            static_cast<const float*>(u), static_cast<float*>(du),
                            static_cast<float*>(dbias), scratch, rows, cols, sums, st);
}

hipError_t bias_dropout_add_fwd(int dtype, const void* in, const void* bias, const void* res,
                                void* out, int rows, int cols, int site, DropoutParams dp,
                                hipStream_t st) {
  const size_t nvec = static_cast<size_t>(rows) * cols / 8;
  const dim3 grid(static_cast<unsigned>((nvec + kThreads - 1) / kThreads));
  const DropoutKey key = make_dropout_key(dp, site);
  if (dtype == 1)
    hipLaunchKernelGGL((bias_dropout_add_kernel<bf16_t>), grid, dim3(kThreads), 0, st,
                       static_cast<const bf16_t*>(in), static_cast<const bf16_t*>(bias),
                       static_cast<const bf16_t*>(res), static_cast<bf16_t*>(out), nvec, cols, key);
  else
    hipLaunchKernelGGL((bias_dropout_add_kernel<float>), grid, dim3(kThreads), 0, st,
                       static_cast<const float*>(in), static_cast<const float*>(bias),
                       static_cast<const float*>(res), static_cast<float*>(out), nvec, cols, key);
  return hipGetLastError();
}

hipError_t dropout_bwd(int dtype, const void* dout, void* din, void* dbias, float* scratch, int rows,
                       int cols, int site, DropoutParams dp, ColumnSums* sums, hipStream_t st) {
  const DropoutKey key = make_dropout_key(dp, site);
  if (dtype == 1) {
    return launch_rows_colsum(DropoutBwdOp<bf16_t>{key}, static_cast<const bf16_t*>(dout),
                              static_cast<const bf16_t*>(nullptr), static_cast<bf16_t*>(din),
                              static_cast<bf16_t*>(dbias), scratch, rows, cols, sums, st);
  }
  return launch_rows_colsum(DropoutBwdOp<float>{key}, static_cast<const float*>(dout),
                            static_cast<const float*>(nullptr), static_cast<float*>(din),
                            static_cast<float*>(dbias), scratch, rows, cols, sums, st);
}

hipError_t column_sum(int dtype, const void* x, void* dbias, float* scratch, int rows, int cols,
                      ColumnSums* sums, hipStream_t st) {
  if (dtype == 1) {
    return launch_rows_colsum(IdentityOp<bf16_t>{}, static_cast<const bf16_t*>(x),
                              static_cast<const bf16_t*>(nullptr), static_cast<bf16_t*>(nullptr),
                              static_cast<bf16_t*>(dbias), scratch, rows, cols, sums, st);
  }
  return launch_rows_colsum(IdentityOp<float>{}, static_cast<const float*>(x),
                            static_cast<const float*>(nullptr), static_cast<float*>(nullptr),
                            static_cast<float*>(dbias), scratch, rows, cols, sums, st);
}

hipError_t dropout_mask_hidden(uint8_t* out, size_t n, int site, DropoutParams dp, hipStream_t st) {
  const size_t ng = n / 8;
  hipLaunchKernelGGL(mask_bytes_kernel, dim3(static_cast<unsigned>((ng + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, st, out, ng, static_cast<uint64_t>(0), make_dropout_key(dp, site));
  return hipGetLastError();
}

hipError_t dropout_mask_attn(uint8_t* out, AttnShape sh, DropoutParams dp, hipStream_t st) {
  // one launch per (bi, hd) slice: slices are contiguous in the output but
  // strided in the global index space when the shard holds a subset of heads
  const size_t slice = static_cast<size_t>(sh.s) * sh.s;
  const size_t ng = slice / 8;
  const DropoutKey key = make_dropout_key(dp, 0);
  for (int bi = 0; bi < sh.b; ++bi)
    for (int hd = 0; hd < sh.a; ++hd) {
      const uint64_t first = (static_cast<uint64_t>(bi) * sh.global_heads + sh.head0 + hd) * slice;
      hipLaunchKernelGGL(mask_bytes_kernel,
                         dim3(static_cast<unsigned>((ng + kThreads - 1) / kThreads)), dim3(kThreads),
                         0, st, out + (static_cast<size_t>(bi) * sh.a + hd) * slice, ng, first / 8,
                         key);
    }
  return hipGetLastError();
}

}  // namespace lynx
