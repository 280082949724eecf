// LayerNorm forward/backward and deterministic column reductions.
//
// These kernels are bound by HBM bandwidth.  A wave owns a row: each lane
// moves 16-byte chunks (8 elements) with consecutive lanes on consecutive
// chunks, so every wave-wide access is one contiguous span; row statistics are
// wave64 butterfly reductions in fp32.
//
// Parameter/bias gradients are sums over all tokens.  They are formed in two
// fixed-order phases (no floating-point atomics): a workgroup owns a segment of
// kReduceRows rows and a 512-column slice, its 4 waves take every 4th row of
// the segment, and their register sums are added in wave order into one
// partial row; reduce_partials then adds the partials in segment order.
#include <algorithm>
#include <atomic>
#include <mutex>

#include "common.h"
#include "kernels.h"

namespace merak {

constexpr int kRowsPerBlock = 4;  // waves per 256-thread workgroup

// Rows of a launch may come from `members` equal groups of mrows rows, group m
// starting m * mstride rows after the pointers given: logical row r is
// physical row (r / mrows) * mstride + r % mrows.
__device__ __forceinline__ int member_row(int r, int mrows, int mstride) {
  return (r / mrows) * mstride + r % mrows;
}

template <typename T, int CH>
__global__ void __launch_bounds__(256) ln_fwd_kernel(int rows, int mrows, int mstride, int h, float eps,
                                                     const T* __restrict__ x,
                                                     const T* __restrict__ gamma, const T* __restrict__ beta,
                                                     T* __restrict__ y, float* __restrict__ mean,
                                                     float* __restrict__ rstd) {
  const int lrow = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (lrow >= rows) return;
  const int row = member_row(lrow, mrows, mstride);
  const T* xr = x + (size_t)row * h;
  float v[CH][8];
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = (lane + 64 * i) * 8;
    if (c < h) {
      load8(xr + c, v[i]);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[i][e];
    }
  }
  const float mu = wave_sum(s) / (float)h;
  float q = 0.0f;
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = (lane + 64 * i) * 8;
    if (c < h) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float d = v[i][e] - mu;
        q += d * d;
      }
    }
  }
  const float var = wave_sum(q) / (float)h;  // biased variance
  const float rs = 1.0f / sqrtf(var + eps);
  T* yr = y + (size_t)row * h;
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = (lane + 64 * i) * 8;
    if (c < h) {
      float g[8], b[8], o[8];
      load8(gamma + c, g);
      load8(beta + c, b);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (v[i][e] - mu) * rs * g[e] + b[e];
      store8(yr + c, o);
    }
  }
  if (lane == 0) {
    mean[row] = mu;
    rstd[row] = rs;
  }
}

// dx = dres + rstd * (dxhat - mean(dxhat) - xhat * mean(dxhat * xhat)),
// dxhat = dout * gamma.  One wave per row; the row stays in registers.
template <typename T, int CH>
__device__ __forceinline__ void ln_bwd_row(int row, int lane, int h, const T* __restrict__ dout,
                                           const T* __restrict__ x, const float* __restrict__ mean,
                                           const float* __restrict__ rstd, const T* __restrict__ gamma,
                                           const T* __restrict__ dres, T* __restrict__ dx) {
  const float mu = mean[row], rs = rstd[row];
  const T* xr = x + (size_t)row * h;
  const T* dr = dout + (size_t)row * h;
  float xh[CH][8], dxh[CH][8];
  float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = (lane + 64 * i) * 8;
    if (c < h) {
      float xv[8], dv[8], g[8];
      load8(xr + c, xv);
      load8(dr + c, dv);
      load8(gamma + c, g);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xh[i][e] = (xv[e] - mu) * rs;
        dxh[i][e] = dv[e] * g[e];
        s1 += dxh[i][e];
        s2 += dxh[i][e] * xh[i][e];
      }
    }
  }
  const float m1 = wave_sum(s1) / (float)h;
  const float m2 = wave_sum(s2) / (float)h;
  const T* rr = dres + (size_t)row * h;
  T* outr = dx + (size_t)row * h;
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    const int c = (lane + 64 * i) * 8;
    if (c < h) {
      float res[8], o[8];
      load8(rr + c, res);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = res[e] + rs * (dxh[i][e] - m1 - xh[i][e] * m2);
      store8(outr + c, o);
    }
  }
}

template <typename T, int CH>
__global__ void __launch_bounds__(256) ln_bwd_kernel(int rows, int mrows, int mstride, int h,
                                                     const T* __restrict__ dout,
                                                     const T* __restrict__ x, const float* __restrict__ mean,
                                                     const float* __restrict__ rstd, const T* __restrict__ gamma,
                                                     const T* __restrict__ dres, T* __restrict__ dx) {
  const int lrow = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
  if (lrow >= rows) return;
  ln_bwd_row<T, CH>(member_row(lrow, mrows, mstride), threadIdx.x & 63, h, dout, x, mean, rstd, gamma, dres, dx);
}

// Segment/slice partial sums.  Mode 0: part0 = sum a.  Mode 1 (LayerNorm
// parameters): part0 = sum a * xhat, part1 = sum a, with xhat rebuilt from x,
// mean and rstd.  One launch covers up to kMaxColJobs reductions; workgroup
// ranges are assigned to the jobs in order.  UNROLL rows of a wave are in flight.
struct ColPartialBatch {
  ColPartialJob j[kMaxColJobs];
  int start[kMaxColJobs + 1];  // first workgroup of each job
  int n;
};

template <typename T, int MODE, int UNROLL = 1>
__device__ __forceinline__ void segment_partials(const ColPartialJob& J, int cx, int seg,
                                                 float (&red)[2][kRowsPerBlock][64 * 8]) {
  constexpr int NQ = MODE == 0 ? 1 : 2;
  const T* __restrict__ a = static_cast<const T*>(J.a);
  const T* __restrict__ x = static_cast<const T*>(J.x);
  const int w = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int c = (cx * 64 + lane) * 8;
  const int r0 = seg * kReduceRows;
  const int r1 = min(r0 + kReduceRows, J.rows);
  float acc[NQ][8];
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[q][e] = 0.0f;
  if (c < J.cols) {
#pragma unroll UNROLL
    for (int r = r0 + w; r < r1; r += kRowsPerBlock) {
      float v[8];
      load8(a + (size_t)r * J.cols + c, v);
      if constexpr (MODE == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[0][e] += v[e];
      } else {
        float xv[8];
        load8(x + (size_t)r * J.cols + c, xv);
        const float mu = J.mean[r], rs = J.rstd[r];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          acc[0][e] += v[e] * ((xv[e] - mu) * rs);
          acc[1][e] += v[e];
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int e = 0; e < 8; ++e) red[q][w][lane * 8 + e] = acc[q][e];
  __syncthreads();
  // 256 threads finish 64 lanes x 8 columns x NQ quantities; wave order fixed.
  for (int idx = threadIdx.x; idx < NQ * 64 * 8; idx += 256) {
    const int q = idx / (64 * 8);
    const int jc = idx % (64 * 8);
    const int col = cx * 64 * 8 + jc;
    if (col < J.cols) {
      float t = 0.0f;
#pragma unroll
      for (int i = 0; i < kRowsPerBlock; ++i) t += red[q][i][jc];
      (q == 0 ? J.p0 : J.p1)[(size_t)seg * J.cols + col] = t;
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) segment_partials_kernel(ColPartialBatch b) {
  __shared__ float red[2][kRowsPerBlock][64 * 8];
  const int bid = blockIdx.x;
  ColPartialJob J = b.j[0];
  int s0 = 0;
#pragma unroll
  for (int i = 1; i < kMaxColJobs; ++i)
    if (i < b.n && bid >= b.start[i]) { J = b.j[i]; s0 = b.start[i]; }
  const int local = bid - s0;
  const int ncx = (J.cols / 8 + 63) / 64;
  if (J.mode == 0) segment_partials<T, 0>(J, local % ncx, local / ncx, red);
  else segment_partials<T, 1>(J, local % ncx, local / ncx, red);
}

// LayerNorm backward and its parameter gradients' partial sums in one launch:
// both read dout and x, and neither needs the other's result.  Each segment of
// kReduceRows rows has kSegRowBlocks row workgroups and one workgroup per 512
// columns of partial sums; a segment's workgroups follow each other on one XCD
// (workgroups go to the 8 XCDs round-robin), so the sums find the rows in its L2
// instead of reading them from memory again.  Bound by memory: 4096 x 3072 in
// bf16 moves 101 MB, 21.4 us (4.7 TB/s, the rate of a large copy); two launches
// took 18.0 + 9.8 us there.  The whole call, with one launch for both final
// sums: 34.5 -> 29.4 us, at 2048 x 1600 21.9 -> 11.7 us.
//
// Above 4096 columns the row workgroups' registers leave one or two waves per
// SIMD, to the workgroups of the partial sums too, which then wait for one row at
// a time: 8192 x 6144 in bf16 took 134 us, with the sums in a launch of their own
// 128.  There they keep four rows (above 6144 columns eight) in flight: 115 us;
// 8192 x 5120 112 -> 98, 12288 x 8192 372 -> 346.  At 4096 columns and fewer,
// with three waves and more, short calls lose 3-5% by it.
constexpr int kSegRowBlocks = kReduceRows / kRowsPerBlock;

template <typename T, int CH>
__global__ void __launch_bounds__(256) ln_bwd_full_kernel(ColPartialJob J, const T* __restrict__ gamma,
                                                          const T* __restrict__ dres, T* __restrict__ dx) {
  constexpr int kUnroll = CH >= 16 ? 8 : CH >= 12 ? 4 : 1;
  __shared__ float red[2][kRowsPerBlock][64 * 8];
  const int ncx = (J.cols / 8 + 63) / 64, per = kSegRowBlocks + ncx;
  const int i = blockIdx.x >> 3, seg = (i / per) * 8 + (blockIdx.x & 7), k = i % per;
  if (seg * kReduceRows >= J.rows) return;
  if (k < kSegRowBlocks) {
    const int row = seg * kReduceRows + k * kRowsPerBlock + (threadIdx.x >> 6);
    if (row < J.rows)
      ln_bwd_row<T, CH>(row, threadIdx.x & 63, J.cols, static_cast<const T*>(J.a), static_cast<const T*>(J.x), J.mean,
                        J.rstd, gamma, dres, dx);
  } else {
    segment_partials<T, 1, kUnroll>(J, k - kSegRowBlocks, seg, red);
  }
}

// out[c] (= or +=) sum_g part[g, c].  16 waves split the groups round-robin and
// their sums are added in wave order, so the result does not depend on timing.
// One launch covers up to kMaxColJobs such sums, 64 columns per workgroup.
constexpr int kReduceWaves = 16;
struct ReduceBatch {
  ReduceJob j[kMaxColJobs];
  int start[kMaxColJobs + 1];
  int n;
};

__global__ void __launch_bounds__(64 * kReduceWaves) reduce_partials_kernel(ReduceBatch b) {
  __shared__ float red[kReduceWaves][64];
  const int bid = blockIdx.x;
  ReduceJob J = b.j[0];
  int s0 = 0;
#pragma unroll
  for (int i = 1; i < kMaxColJobs; ++i)
    if (i < b.n && bid >= b.start[i]) { J = b.j[i]; s0 = b.start[i]; }
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int c = (bid - s0) * 64 + lane;
  float s = 0.0f;
  if (c < J.cols)
    for (int g = w; g < J.groups; g += kReduceWaves) s += J.part[(size_t)g * J.cols + c];
  red[w][lane] = s;
  __syncthreads();
  if (w == 0 && c < J.cols) {
    float t = 0.0f;
#pragma unroll
    for (int i = 0; i < kReduceWaves; ++i) t += red[i][lane];
    J.out[c] = J.accumulate ? J.out[c] + t : t;
  }
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
// Rows of one launch: `rows` logical rows in groups of mrows, mstride apart.
struct RowMap {
  int rows, mrows, mstride;
};

template <typename T, int CH>
static hipError_t ln_fwd_t(RowMap rm, int h, float eps, const void* x, const void* g, const void* b, void* y,
                           float* mean, float* rstd, hipStream_t s) {
  dim3 grid((rm.rows + kRowsPerBlock - 1) / kRowsPerBlock);
  hipLaunchKernelGGL((ln_fwd_kernel<T, CH>), grid, dim3(256), 0, s, rm.rows, rm.mrows, rm.mstride, h, eps,
                     (const T*)x, (const T*)g, (const T*)b, (T*)y, mean, rstd);
  return hipGetLastError();
}

template <typename T>
static hipError_t ln_fwd_dispatch(RowMap rm, int h, float eps, const void* x, const void* g, const void* b,
                                  void* y, float* mean, float* rstd, hipStream_t s) {
  const int ch = (h + 511) / 512;
  if (ch <= 1) return ln_fwd_t<T, 1>(rm, h, eps, x, g, b, y, mean, rstd, s);
  if (ch <= 2) return ln_fwd_t<T, 2>(rm, h, eps, x, g, b, y, mean, rstd, s);
  if (ch <= 4) return ln_fwd_t<T, 4>(rm, h, eps, x, g, b, y, mean, rstd, s);
  if (ch <= 6) return ln_fwd_t<T, 6>(rm, h, eps, x, g, b, y, mean, rstd, s);
  if (ch <= 8) return ln_fwd_t<T, 8>(rm, h, eps, x, g, b, y, mean, rstd, s);
  if (ch <= 12) return ln_fwd_t<T, 12>(rm, h, eps, x, g, b, y, mean, rstd, s);
  if (ch <= 16) return ln_fwd_t<T, 16>(rm, h, eps, x, g, b, y, mean, rstd, s);
  return hipErrorInvalidValue;
}

static bool row_map(int rows, int members, int member_stride, RowMap* rm) {
  if (members < 1 || (members > 1 && member_stride < rows)) return false;
  if ((long long)rows * members > 0x7fffffffLL || (long long)member_stride * (members - 1) + rows > 0x7fffffffLL)
    return false;
  *rm = {rows * members, rows, members > 1 ? member_stride : rows};
  return true;
}

hipError_t launch_layernorm_fwd(int dtype, int rows, int h, float eps, const void* x, const void* gamma,
                                const void* beta, void* y, float* mean, float* rstd, hipStream_t stream,
                                int members, int member_stride) {
  if (rows <= 0) return hipSuccess;
  RowMap rm;
  if (h % 8 != 0 || !row_map(rows, members, member_stride, &rm)) return hipErrorInvalidValue;
  return dtype == DT_BF16 ? ln_fwd_dispatch<bf16_t>(rm, h, eps, x, gamma, beta, y, mean, rstd, stream)
                          : ln_fwd_dispatch<float>(rm, h, eps, x, gamma, beta, y, mean, rstd, stream);
}

template <typename T, int CH>
static hipError_t ln_bwd_t(RowMap rm, int h, const void* dout, const void* x, const float* mean,
                           const float* rstd, const void* g, const void* dres, void* dx, hipStream_t s) {
  dim3 grid((rm.rows + kRowsPerBlock - 1) / kRowsPerBlock);
  hipLaunchKernelGGL((ln_bwd_kernel<T, CH>), grid, dim3(256), 0, s, rm.rows, rm.mrows, rm.mstride, h,
                     (const T*)dout, (const T*)x, mean, rstd, (const T*)g, (const T*)dres, (T*)dx);
  return hipGetLastError();
}

template <typename T>
static hipError_t ln_bwd_dispatch(RowMap rm, int h, const void* dout, const void* x, const float* mean,
                                  const float* rstd, const void* g, const void* dres, void* dx, hipStream_t s) {
  const int ch = (h + 511) / 512;
  if (ch <= 1) return ln_bwd_t<T, 1>(rm, h, dout, x, mean, rstd, g, dres, dx, s);
  if (ch <= 2) return ln_bwd_t<T, 2>(rm, h, dout, x, mean, rstd, g, dres, dx, s);
  if (ch <= 4) return ln_bwd_t<T, 4>(rm, h, dout, x, mean, rstd, g, dres, dx, s);
  if (ch <= 6) return ln_bwd_t<T, 6>(rm, h, dout, x, mean, rstd, g, dres, dx, s);
  if (ch <= 8) return ln_bwd_t<T, 8>(rm, h, dout, x, mean, rstd, g, dres, dx, s);
  if (ch <= 12) return ln_bwd_t<T, 12>(rm, h, dout, x, mean, rstd, g, dres, dx, s);
  if (ch <= 16) return ln_bwd_t<T, 16>(rm, h, dout, x, mean, rstd, g, dres, dx, s);
  return hipErrorInvalidValue;
}

hipError_t launch_layernorm_bwd(int dtype, int rows, int h, const void* dout, const void* x, const float* mean,
                                const float* rstd, const void* gamma, const void* dres, void* dx,
                                hipStream_t stream, int members, int member_stride) {
  if (rows <= 0) return hipSuccess;
  RowMap rm;
  if (h % 8 != 0 || !row_map(rows, members, member_stride, &rm)) return hipErrorInvalidValue;
  return dtype == DT_BF16 ? ln_bwd_dispatch<bf16_t>(rm, h, dout, x, mean, rstd, gamma, dres, dx, stream)
                          : ln_bwd_dispatch<float>(rm, h, dout, x, mean, rstd, gamma, dres, dx, stream);
}

template <typename T, int CH>
static hipError_t ln_bwd_full_t(const ColPartialJob& J, const void* g, const void* dres, void* dx, hipStream_t s) {
  const long long segs = ((long long)reduce_groups(J.rows) + 7) / 8 * 8;
  const long long wg = segs * (kSegRowBlocks + (J.cols / 8 + 63) / 64);
  if (wg > 0x7fffffffLL) return hipErrorInvalidValue;
  hipLaunchKernelGGL((ln_bwd_full_kernel<T, CH>), dim3((unsigned)wg), dim3(256), 0, s, J, (const T*)g, (const T*)dres,
                     (T*)dx);
  return hipGetLastError();
}

template <typename T>
static hipError_t ln_bwd_full_dispatch(const ColPartialJob& J, const void* g, const void* dres, void* dx,
                                       hipStream_t s) {
  const int ch = (J.cols + 511) / 512;
  if (ch <= 1) return ln_bwd_full_t<T, 1>(J, g, dres, dx, s);
  if (ch <= 2) return ln_bwd_full_t<T, 2>(J, g, dres, dx, s);
  if (ch <= 4) return ln_bwd_full_t<T, 4>(J, g, dres, dx, s);
  if (ch <= 6) return ln_bwd_full_t<T, 6>(J, g, dres, dx, s);
  if (ch <= 8) return ln_bwd_full_t<T, 8>(J, g, dres, dx, s);
  if (ch <= 12) return ln_bwd_full_t<T, 12>(J, g, dres, dx, s);
  if (ch <= 16) return ln_bwd_full_t<T, 16>(J, g, dres, dx, s);
  return hipErrorInvalidValue;
}

hipError_t launch_layernorm_bwd_full(int dtype, int rows, int h, const void* dout, const void* x, const float* mean,
                                     const float* rstd, const void* gamma, const void* dres, void* dx, float* dgamma,
                                     float* dbeta, int accumulate, float* part, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  if (h <= 0 || h % 8 != 0) return hipErrorInvalidValue;
  float* part_b = part + reduce_groups(rows) * (size_t)h;
  const ColPartialJob J{1, rows, h, dout, x, mean, rstd, part, part_b};
  hipError_t e = dtype == DT_BF16 ? ln_bwd_full_dispatch<bf16_t>(J, gamma, dres, dx, stream)
                                  : ln_bwd_full_dispatch<float>(J, gamma, dres, dx, stream);
  if (e != hipSuccess) return e;
  const int G = (int)reduce_groups(rows);
  const ReduceJob rj[2] = {{G, h, part, dgamma, accumulate}, {G, h, part_b, dbeta, accumulate}};
  return launch_reduce_partials_batch(rj, 2, stream);
}

hipError_t launch_column_partials_batch(int dtype, const ColPartialJob* jobs, int n, hipStream_t stream) {
  if (n < 1 || n > kMaxColJobs) return hipErrorInvalidValue;
  ColPartialBatch b;
  b.n = 0;
  int total = 0;
  for (int i = 0; i < n; ++i) {
    const ColPartialJob& J = jobs[i];
    if (J.rows <= 0 || J.cols <= 0) continue;
    if (J.cols % 8 != 0 || (J.mode != 0 && J.mode != 1)) return hipErrorInvalidValue;
    const long long wg = (long long)((J.cols / 8 + 63) / 64) * (long long)reduce_groups(J.rows);
    if (total + wg > 0x7fffffffLL) return hipErrorInvalidValue;
    b.j[b.n] = J;
    b.start[b.n] = total;
    total += (int)wg;
    ++b.n;
  }
  if (b.n == 0) return hipSuccess;
  b.start[b.n] = total;
  if (dtype == DT_BF16)
    hipLaunchKernelGGL(segment_partials_kernel<bf16_t>, dim3(total), dim3(256), 0, stream, b);
  else
    hipLaunchKernelGGL(segment_partials_kernel<float>, dim3(total), dim3(256), 0, stream, b);
  return hipGetLastError();
}

hipError_t launch_column_partials(int dtype, int rows, int cols, const void* x, float* part, hipStream_t stream) {
  const ColPartialJob j{0, rows, cols, x, nullptr, nullptr, nullptr, part, nullptr};
  return launch_column_partials_batch(dtype, &j, 1, stream);
}

hipError_t launch_reduce_partials_batch(const ReduceJob* jobs, int n, hipStream_t stream) {
  if (n < 1 || n > kMaxColJobs) return hipErrorInvalidValue;
  ReduceBatch b;
  b.n = 0;
  int total = 0;
  for (int i = 0; i < n; ++i) {
    if (jobs[i].cols <= 0) continue;
    b.j[b.n] = jobs[i];
    b.start[b.n] = total;
    total += (jobs[i].cols + 63) / 64;
    ++b.n;
  }
  if (b.n == 0) return hipSuccess;
  b.start[b.n] = total;
  hipLaunchKernelGGL(reduce_partials_kernel, dim3(total), dim3(64 * kReduceWaves), 0, stream, b);
  return hipGetLastError();
}

hipError_t launch_reduce_partials(int groups, int cols, const float* part, float* out, int accumulate,
                                  hipStream_t stream) {
  const ReduceJob j{groups, cols, part, out, accumulate};
  return launch_reduce_partials_batch(&j, 1, stream);
}

// ---------------------------------------------------------------------------
// Scratch of the allocation-free LayerNorm backward: a fixed-size array in the
// library's own device memory, one copy per GPU, held until the process ends.
// The host never passes the array's name to a kernel (on the host it stands
// for a host-side shadow): its device address is taken once per device with
// hipGetSymbolAddress and kept per device.
// ---------------------------------------------------------------------------
static __device__ __align__(256) float scratch[kNoAllocScratchFloats];

// ---------------------------------------------------------------------------
// Non-finite scan (failure detection): an element is NaN or +-Inf iff its
// exponent field is all ones (bf16: bits 7..14, fp32: bits 23..30).
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned nonfinite_bf16_pair(uint32_t w) {
  return ((w & 0x7f80u) == 0x7f80u) + ((w & 0x7f800000u) == 0x7f800000u);
}
__device__ __forceinline__ unsigned nonfinite_f32(uint32_t w) { return (w & 0x7f800000u) == 0x7f800000u; }

__global__ void __launch_bounds__(64) zero_count_kernel(unsigned long long* count) {
  if (threadIdx.x == 0) *count = 0ull;
}

// Grid-stride over 16-byte chunks; the elements past the last whole chunk are
// taken by workgroup 0.  Per-thread counts are summed in LDS, then one atomic
// add per workgroup: an integer sum, so the result does not depend on order.
template <bool BF16>
__global__ void __launch_bounds__(256) count_nonfinite_kernel(const uint32_t* __restrict__ x, long long n,
                                                              unsigned long long* __restrict__ count) {
  __shared__ unsigned long long blk;
  constexpr int PER = BF16 ? 8 : 4;  // elements per 16-byte chunk
  const long long chunks = n / PER;
  unsigned long long c = 0;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < chunks; i += stride) {
    const u32x4_t w = reinterpret_cast<const u32x4_t*>(x)[i];
#pragma unroll
    for (int e = 0; e < 4; ++e) c += BF16 ? nonfinite_bf16_pair(w[e]) : nonfinite_f32(w[e]);
  }
  if (blockIdx.x == 0) {
    for (long long i = chunks * PER + threadIdx.x; i < n; i += blockDim.x) {
      if constexpr (BF16) {
        const uint16_t v = reinterpret_cast<const uint16_t*>(x)[i];
        c += (v & 0x7f80u) == 0x7f80u;
      } else {
        c += nonfinite_f32(x[i]);
      }
    }
  }
  if (threadIdx.x == 0) blk = 0ull;
  __syncthreads();
  if (c) atomicAdd(&blk, c);
  __syncthreads();
  if (threadIdx.x == 0 && blk) atomicAdd(count, blk);
}

hipError_t launch_count_nonfinite(int dtype, const void* x, long long n, unsigned long long* count,
                                  hipStream_t stream) {
  hipLaunchKernelGGL(zero_count_kernel, dim3(1), dim3(64), 0, stream, count);
  if (n <= 0) return hipGetLastError();
  const long long chunks = n / (dtype == DT_BF16 ? 8 : 4);
  const long long blocks = std::min<long long>(std::max<long long>((chunks + 255) / 256, 1), 2048);
  if (dtype == DT_BF16)
    hipLaunchKernelGGL((count_nonfinite_kernel<true>), dim3((unsigned)blocks), dim3(256), 0, stream,
                       (const uint32_t*)x, n, count);
  else
    hipLaunchKernelGGL((count_nonfinite_kernel<false>), dim3((unsigned)blocks), dim3(256), 0, stream,
                       (const uint32_t*)x, n, count);
  return hipGetLastError();
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
std::atomic<float*> g_scratch_ptr[kMaxDevices];
}  // namespace

hipError_t noalloc_scratch(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  float* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    p = g_scratch_ptr[dev].load(std::memory_order_relaxed);
    if (!p) {
      void* addr = nullptr;
      e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
      if (e != hipSuccess) return e;
      if (!addr) return hipErrorInvalidSymbol;
      p = static_cast<float*>(addr);
      g_scratch_ptr[dev].store(p, std::memory_order_release);
    }
  }
  *out = p;
  return hipSuccess;
}

}  // namespace merak
