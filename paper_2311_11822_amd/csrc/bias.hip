// Bias gradients (appendix A.1 of the paper, last paragraph): the per-sample bias gradient is
// 1^T dL/ds_i, the sum of sample i's T output-gradient rows; its norm is taken by
// instantiation.  The B x d_out matrix of these sums is tiny, so it is kept (book-keeping): the
// clipped bias gradient sum_i C_i 1^T g_i is then formed from it without reading g again.
// The kernels are streams over memory (HBM-bound) or, for small samples, latency-bound; sums run in a fixed order.
#include <algorithm>
#include <type_traits>

#include "dp_internal.h"

namespace dpbk {

namespace {

constexpr int kRowGroups = 16, kColThreads = 32;

// One workgroup: sample blockIdx.y, a strip of 32 * VEC columns.  Thread (rg, ct) adds rows
// rg, rg + 16, ... of its VEC columns; the 16 row groups are then added in order through LDS.
template <int DT>                       // dp_dtype of g
__global__ void __launch_bounds__(kRowGroups * kColThreads)
bias_colsum_kernel(const void* __restrict__ g_all, int T, int p, float* __restrict__ colsum) {
  constexpr bool HALF = DT != DP_F32;   // 16-bit storage: 8 columns per thread
  constexpr int VEC = HALF ? 8 : 1;
  __shared__ float red[kRowGroups][kColThreads * VEC + 1];
  const int ct = threadIdx.x % kColThreads, rg = threadIdx.x / kColThreads;
  const int i = blockIdx.y;
  const int col = (blockIdx.x * kColThreads + ct) * VEC;
  float acc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) acc[v] = 0.f;
  if (col < p) {
    if (HALF) {
      const uint16_t* g = static_cast<const uint16_t*>(g_all) + (size_t)i * T * p + col;
      auto add = [&](const uint4& w) {
        const uint32_t u[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (DT == DP_BF16) {
            acc[2 * q] += __uint_as_float(u[q] << 16);             // bf16 -> fp32 is a shift
            acc[2 * q + 1] += __uint_as_float(u[q] & 0xFFFF0000u);
          } else {
            acc[2 * q] += (float)__builtin_bit_cast(_Float16, (uint16_t)(u[q] & 0xFFFFu));
            acc[2 * q + 1] += (float)__builtin_bit_cast(_Float16, (uint16_t)(u[q] >> 16));
          }
        }
      };
      // four rows in flight per thread; they are added in row order, so the sum does not depend
      // on the unrolling
      int t = rg;
      for (; t + 3 * kRowGroups < T; t += 4 * kRowGroups) {
        uint4 w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) w[u] = *reinterpret_cast<const uint4*>(g + (size_t)(t + u * kRowGroups) * p);
#pragma unroll
        for (int u = 0; u < 4; ++u) add(w[u]);
      }
      for (; t < T; t += kRowGroups) add(*reinterpret_cast<const uint4*>(g + (size_t)t * p));
    } else {
      const float* g = static_cast<const float*>(g_all) + (size_t)i * T * p + col;
      for (int t = rg; t < T; t += kRowGroups) acc[0] += g[(size_t)t * p];
    }
  }
#pragma unroll
  for (int v = 0; v < VEC; ++v) red[rg][ct * VEC + v] = acc[v];
  __syncthreads();
  for (int c = threadIdx.x; c < kColThreads * VEC; c += kRowGroups * kColThreads) {
    const int out_col = blockIdx.x * kColThreads * VEC + c;
    if (out_col < p) {
      float s = 0.f;
#pragma unroll
      for (int r = 0; r < kRowGroups; ++r) s += red[r][c];
      colsum[(size_t)i * p + out_col] = s;
    }
  }
}

// The same of few or small strips, 64 columns each, where the kernel above is a chain of memory latencies in few workgroups:
// thread (rg, ct) adds rows rg, rg + groups, ... of its 8 columns, ROWS rows in flight, and groups of eight row groups are
// added up side by side.  A whole dp_bias_norm, us, 256-column strips and these: 8 x 128 tokens of 768 columns 5.33, 4.83; of 3072
// 5.71, 5.56; 16 x 256 x 768 6.33, 5.42; 8 x 512 x 1280 9.3, 6.5; 1 x 512 x 1024 7.4, 4.5; 2 x 4096 x 768 45.8, 17.1; what streams
// prefers the long rows: 16 x 256 x 3072 9.0, 9.7; 8 x 512 x 5120 12.4, 14.1.
template <int DT, int THREADS, int ROWS>
__global__ void __launch_bounds__(THREADS)
bias_colsum_few_kernel(const uint16_t* __restrict__ g_all, int T, int p, float* __restrict__ colsum) {
  constexpr int GROUPS = THREADS / 8, PARTS = GROUPS / 8;
  __shared__ float red[GROUPS][65];
  __shared__ float sub[PARTS][64];
  const int ct = threadIdx.x & 7, rg = threadIdx.x >> 3, i = blockIdx.y;
  const int col = blockIdx.x * 64 + ct * 8;
  float acc[8] = {};
  if (col < p) {
    const uint16_t* g = g_all + (size_t)i * T * p + col;
    for (unsigned t0 = rg; t0 < (unsigned)T; t0 += ROWS * GROUPS) {
      uint4 w[ROWS];
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        const unsigned t = t0 + u * GROUPS;
        w[u] = make_uint4(0, 0, 0, 0);
        if (t < (unsigned)T) w[u] = *reinterpret_cast<const uint4*>(g + (size_t)t * p);
      }
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        const uint32_t x[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t pair = x[k / 2];
          if (DT == DP_BF16)
            acc[k] += __uint_as_float(k & 1 ? pair & 0xFFFF0000u : pair << 16);      // bf16 -> fp32 is a shift
          else
            acc[k] += (float)__builtin_bit_cast(_Float16, (uint16_t)(k & 1 ? pair >> 16 : pair & 0xFFFFu));
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) red[rg][8 * ct + k] = acc[k];
  __syncthreads();
  const int c = threadIdx.x & 63, part = threadIdx.x >> 6;
  float s = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) s += red[8 * part + r][c];
  sub[part][c] = s;
  __syncthreads();
  if (part == 0 && blockIdx.x * 64 + c < (unsigned)p) {
    float total = 0.f;
#pragma unroll
    for (int r = 0; r < PARTS; ++r) total += sub[r][c];
    colsum[(size_t)i * p + blockIdx.x * 64 + c] = total;
  }
}

// Strips of 64 columns: few of them, or not many, of few values in all and of whole 128-byte lines (both sides beside the kernel;
// 50 x 20 x 5000, 3950 strips, 7.7 and 8.4; 55 x 136 x 696, rows of 1392 bytes, 7.1 and 7.9).
constexpr int64_t kFewStrips = 256, kMostStrips = 1280, kFewValues = 6 << 20;
bool few_strips(int B, int64_t T, int p) {
  const int64_t strips = ((int64_t)p + 63) / 64 * B;
  return strips <= kFewStrips || (p % 64 == 0 && strips <= kMostStrips && T * p <= kFewValues / B);
}

// Column sums and their norm in one launch, one workgroup to a sample, where that is no slower than two: a launch costs
// the host 2.4 us, and a workgroup of 1024 threads that has eight loads of each in flight reads 90 GB/s.  Thread (rg, ct)
// adds rows rg, rg + groups, ... of its 8 columns, eight rows in flight and added in pairs; the row groups are added
// through LDS.  Times on the GPU, us, here and in two launches (8 samples): 16 tokens of 768 columns 3.7 and 4.9,
// 160 x 256 4.1 and 5.2, 16 x 3072 4.9 and 5.1, 1 x 8192 5.8 and 5.6, 160 x 512 5.5 and 5.3, 128 x 1536 7.2 and 5.1.  Up to
// 256 columns the two-launch form has one workgroup to a sample too, of a quarter of the loads in flight: 2048 x 64 6.4
// and 11.5, 2048 x 200 10.9 and 12.0.
// A workgroup has 64, 256 or 1024 threads, as many as have rows to load or a column to add up (the sums are the same):
// with 1024 for any sample, many small ones wait for waves with nothing to do (65535 samples of 1 x 64: 228 us, 168 in
// two launches, now 29; 4096 of 16 x 256 18.4, 16.1, 8.3).
constexpr int kOneThreads = 1024, kOneRows = 8;
template <int DT, int THREADS>
__global__ void __launch_bounds__(THREADS)
bias_norm_kernel(const uint16_t* __restrict__ g_all, int T, int p, float* __restrict__ colsum, float* __restrict__ sqnorm) {
  __shared__ float red[THREADS * 8];
  __shared__ float wave_sum[THREADS / 64];
  const int tid = threadIdx.x, i = blockIdx.x;
  const int chunks = p / 8;
  const int groups = min(kOneThreads / chunks, (T - 1) / kOneRows + 1);      // of all sizes: the same sums
  const int rg = tid / chunks, ct = tid - rg * chunks;
  if (rg < groups) {
    const uint16_t* g = g_all + (size_t)i * T * p + 8 * ct;
    float acc[8] = {};
    for (unsigned t0 = rg; t0 < (unsigned)T; t0 += kOneRows * groups) {
      uint4 w[kOneRows];
#pragma unroll
      for (int u = 0; u < kOneRows; ++u) {
        const unsigned t = min(t0 + u * groups, (unsigned)T - 1);
        w[u] = *reinterpret_cast<const uint4*>(g + (size_t)t * p);
      }
#pragma unroll
      for (int u = 0; u < kOneRows; ++u)
        if (t0 + u * groups >= (unsigned)T) w[u] = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        float v[kOneRows];
#pragma unroll
        for (int u = 0; u < kOneRows; ++u) {
          const uint32_t x[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
          const uint32_t pair = x[k / 2];
          if (DT == DP_BF16)
            v[u] = __uint_as_float(k & 1 ? pair & 0xFFFF0000u : pair << 16);      // bf16 -> fp32 is a shift
          else
            v[u] = (float)__builtin_bit_cast(_Float16, (uint16_t)(k & 1 ? pair >> 16 : pair & 0xFFFFu));
        }
        acc[k] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
      }
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) red[rg * p + 8 * ct + k] = acc[k];
  }
  __syncthreads();
  float s = 0.f;
  for (int c = tid; c < p; c += THREADS) {
    float part[4] = {};
    int r = 0;
    for (; r + 4 <= groups; r += 4)
#pragma unroll
      for (int q = 0; q < 4; ++q) part[q] += red[(r + q) * p + c];
    for (; r < groups; ++r) part[r & 3] += red[r * p + c];
    const float v = (part[0] + part[1]) + (part[2] + part[3]);
    colsum[(size_t)i * p + c] = v;
    s = fmaf(v, v, s);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((tid & 63) == 0) wave_sum[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) {
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) total += wave_sum[w];
    sqnorm[i] = total;
  }
}

// These two kernels move a few hundred KiB at most: what bounds them is the chain of memory latencies of a
// thread, so every thread asks for all it needs at once.  (One load after the other, the square
// sum took 4.1 us and the weighted sum 4.8 us for 8 x 768 .. 3072 values; so 2.7 and 3.3.)

// sqnorm[i] = sum_k colsum[i,k]^2; one workgroup per sample, fixed-order reduction.
constexpr int kSqThreads = 512, kSqBatch = 8;
__global__ void __launch_bounds__(kSqThreads)
bias_sqnorm_kernel(const float* __restrict__ colsum, int p, float* __restrict__ sqnorm) {
  __shared__ float red[kSqThreads / 64];
  const float* row = colsum + (size_t)blockIdx.x * p;
  float s = 0.f;
  // unsigned: the last round's columns may lie past INT32_MAX
  for (unsigned k0 = threadIdx.x; k0 < (unsigned)p; k0 += kSqBatch * kSqThreads) {
    float v[kSqBatch];
#pragma unroll
    for (int q = 0; q < kSqBatch; ++q) {
      const unsigned k = k0 + q * kSqThreads;
      v[q] = k < (unsigned)p ? row[k] : 0.f;
    }
#pragma unroll
    for (int q = 0; q < kSqBatch; ++q) s = fmaf(v[q], v[q], s);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < kSqThreads / 64; ++w) total += red[w];
    sqnorm[blockIdx.x] = total;
  }
}

// grad_b[k] (+)= sum_i C_i colsum[i,k]; small workgroups, so that a few hundred columns use several compute units
constexpr int kSumThreads = 64, kSumBatch = 16;
__global__ void __launch_bounds__(kSumThreads)
clipped_bias_kernel(const float* __restrict__ colsum, int B, int p, const float* __restrict__ C,
                    float* __restrict__ grad_b, int accumulate) {
  const int k = blockIdx.x * kSumThreads + threadIdx.x;
  if (k >= p) return;
  const float old = accumulate ? grad_b[k] : 0.f;
  float s = 0.f;
  for (unsigned i0 = 0; i0 < (unsigned)B; i0 += kSumBatch) {
    float c[kSumBatch], v[kSumBatch];
#pragma unroll
    for (int q = 0; q < kSumBatch; ++q) {
      const unsigned i = min(i0 + q, (unsigned)B - 1);
      c[q] = C[i];
      v[q] = colsum[(size_t)i * p + k];
    }
#pragma unroll
    for (int q = 0; q < kSumBatch; ++q)
      if (i0 + q < (unsigned)B) s = fmaf(c[q], v[q], s);
  }
  grad_b[k] = accumulate ? old + s : s;
}

// One launch?  Near the lines (160 x 512 values, one row of 8192) it takes 0.2 to 0.4 us more on the GPU for the host's 2.4.
// Many samples of 129 to 256 columns that take a thread more than one trip stream better in the other form (256 x 1024
// tokens of 256 columns: 27.7 and 22.8 us, 2048 x 1024 207 and 188; of 200 columns, 512 x 1024: the same).
constexpr int kOneColumns = 256, kOneValues = 160 * 512, kManySamples = 256;
bool one_launch(int B, int64_t T, int p) {
  if (T * p <= kOneValues) return p <= 8 * kOneThreads;
  return p <= kOneColumns && (p <= kOneColumns / 2 || B < kManySamples);
}

}  // namespace

dp_status launch_bias_norm(const void* g, dp_dtype dt, int B, int T, int p, float* colsum,
                           float* sqnorm_out, hipStream_t s) {
  if (dt != DP_F32 && one_launch(B, T, p)) {
    const int need = std::max(std::min(kOneThreads / (p / 8), (T - 1) / kOneRows + 1) * (p / 8), p);
    auto launch = [&](auto threads_tag) {
      constexpr int THREADS = decltype(threads_tag)::value;
      auto kernel = dt == DP_BF16 ? bias_norm_kernel<DP_BF16, THREADS> : bias_norm_kernel<DP_F16, THREADS>;
      hipLaunchKernelGGL(kernel, dim3(B), dim3(THREADS), 0, s, static_cast<const uint16_t*>(g), T, p, colsum, sqnorm_out);
    };
    if (need <= 64)
      launch(std::integral_constant<int, 64>{});
    else if (need <= 256)
      launch(std::integral_constant<int, 256>{});
    else
      launch(std::integral_constant<int, kOneThreads>{});
    return hip_status(hipGetLastError());
  }
  if (dt != DP_F32 && few_strips(B, T, p)) {
    auto launch = [&](auto threads_tag, auto rows_tag) {
      constexpr int THREADS = decltype(threads_tag)::value, ROWS = decltype(rows_tag)::value;
      auto kernel = dt == DP_BF16 ? bias_colsum_few_kernel<DP_BF16, THREADS, ROWS> : bias_colsum_few_kernel<DP_F16, THREADS, ROWS>;
      hipLaunchKernelGGL(kernel, dim3((p + 63u) / 64, B), dim3(THREADS), 0, s, static_cast<const uint16_t*>(g), T, p, colsum);
    };
    using std::integral_constant;
    if (T <= 128)                                        // one trip
      launch(integral_constant<int, 256>{}, integral_constant<int, 4>{});
    else if (T <= 256)
      launch(integral_constant<int, 512>{}, integral_constant<int, 4>{});
    else
      launch(integral_constant<int, 512>{}, integral_constant<int, 8>{});
    if (hipGetLastError() != hipSuccess) return DP_ERR_HIP;
    hipLaunchKernelGGL(bias_sqnorm_kernel, dim3(B), dim3(kSqThreads), 0, s, colsum, p, sqnorm_out);
    return hip_status(hipGetLastError());
  }
  const int cols_per_block = kColThreads * (dt == DP_F32 ? 1 : 8);
  const dim3 grid((p + cols_per_block - 1) / cols_per_block, B), block(kRowGroups * kColThreads);
  if (dt == DP_BF16)
    hipLaunchKernelGGL(bias_colsum_kernel<DP_BF16>, grid, block, 0, s, g, T, p, colsum);
  else if (dt == DP_F16)
    hipLaunchKernelGGL(bias_colsum_kernel<DP_F16>, grid, block, 0, s, g, T, p, colsum);
  else
    hipLaunchKernelGGL(bias_colsum_kernel<DP_F32>, grid, block, 0, s, g, T, p, colsum);
  if (hipGetLastError() != hipSuccess) return DP_ERR_HIP;
  hipLaunchKernelGGL(bias_sqnorm_kernel, dim3(B), dim3(kSqThreads), 0, s, colsum, p, sqnorm_out);
  return hip_status(hipGetLastError());
}

dp_status launch_clipped_bias_grad(const float* colsum, int B, int p, const float* C, float* grad_b,
                                   int accumulate, hipStream_t s) {
  hipLaunchKernelGGL(clipped_bias_kernel, dim3((p + kSumThreads - 1) / kSumThreads), dim3(kSumThreads), 0, s, colsum,
                     B, p, C, grad_b, accumulate);
  return hip_status(hipGetLastError());
}

}  // namespace dpbk
