// Ghost norm of short samples (appendix A.1 of the paper, right side of eq. "mixed ghost norm"), up to
// 32 tokens:   sqnorm[i] = sum_{t,t'} (a_t . a_t') (g_t . g_t').
//
// A sample of T tokens fills T of the 32 rows of a matrix instruction, and the kernels that give a
// sample a workgroup and a 128- or 256-row tile spend their time on LDS traffic for rows that are
// not there (measured at T = 1, d = 1024: 437 us for 512 samples x 8 layers whose a and g take 7 us to read).
// Here one workgroup takes the 32 / T consecutive samples that fit 32 rows, which are consecutive rows
// in memory too: one 32 x 32 Gram matrix per operand, of which the T x T blocks on the diagonal count. Both
// operands of a x x^T product are the same registers, loaded straight from global memory (a lane's
// 16 bytes are eight consecutive columns of one row), so nothing is staged; the eight waves take every eighth
// 16-column step and add their parts in LDS in a fixed order.  What bounds it is the read of a and g.
// The squared norms are final: no per-tile partial sums, no launch that adds them.
// Where few workgroups would leave compute units idle, each takes a half, a quarter ... of those samples, at the rows that
// they have in any case, so that the bits do not depend on it: a workgroup of this kernel, which waits for its
// loads before it multiplies, reads no more than 24 to 30 GB/s.
// 512 samples of one token, eight layers 1024 x 1024 .. 4096, with 128 and 256 workgroups: 14.1 -> 10.2 us.
#include <algorithm>

#include "clip.h"
#include "dp_internal.h"

namespace dpbk {

namespace {

constexpr int kWaves = 8, kThreads = 64 * kWaves, kRows = 32;
constexpr int kDepth = 8;                        // 16-byte loads in flight per lane

// This wave's part of the Gram matrix of the 32 rows at x (those with `valid` lanes; the others count as zeros).
template <bool F16>
__device__ __forceinline__ f32x16 gram_part(const uint16_t* x, int width, bool valid, int wave, int lane) {
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  const uint16_t* row = x + (size_t)(lane & 31) * width;
  for (int k0 = wave * 16; k0 < width; k0 += kDepth * kWaves * 16) {
    bf16x8 f[kDepth];
#pragma unroll
    for (int q = 0; q < kDepth; ++q) {
      const int k = k0 + q * kWaves * 16 + 8 * (lane >> 5);
      uint4 w = make_uint4(0, 0, 0, 0);
      if (valid && k < width) w = *reinterpret_cast<const uint4*>(row + k);
      f[q] = __builtin_bit_cast(bf16x8, w);
    }
#pragma unroll
    for (int q = 0; q < kDepth; ++q) acc = mfma16<F16>(f[q], f[q], acc);
  }
  return acc;
}

template <bool F16>
__global__ void __launch_bounds__(kThreads)
ghost_brief_kernel(const GroupArgs ga, float* sqnorm, const NormClip nc, int first) {
  __shared__ float part_a[kWaves][16][64], part_g[kWaves][16][64];       // 64 KiB: two workgroups per compute unit
  const int block = first + blockIdx.x;
  const int l = layer_of(ga, block);
  const GroupLayer& ly = ga.layer[l];
  const int T = ly.T, per = kRows / T, parts = ly.tiles_per_sample;
  int rows32 = block - ly.tile_begin, begin = 0, end = per;                  // which 32 rows; this workgroup's samples
  // Launches of more than 256 workgroups have one to 32 rows.  The quotients are of numbers below 512 by up to 32 (integer
  // divisions cost 0.1 us: two samples of 32 tokens, 24 layers 128 x 384 5.0 -> 4.8 us, 3000 of ten tokens 18.7 -> 17.9).
  if (parts > 1) {
    const float inv = __builtin_amdgcn_rcpf((float)parts);
    const int slots = min(per, ga.B);                                        // of 32 rows that hold a sample
    const int share = (int)(((float)(slots + parts - 1) + 0.5f) * inv), local = rows32;
    rows32 = (int)(((float)local + 0.5f) * inv);
    begin = (local - rows32 * parts) * share;
    end = min(begin + share, slots);
  }
  const int i0 = rows32 * per;                                               // first sample of the 32 rows
  end = min(end, ga.B - i0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool valid = (lane & 31) >= begin * T && (lane & 31) < end * T;
  const size_t row0 = (size_t)i0 * T;
  const f32x16 xa = gram_part<F16>(static_cast<const uint16_t*>(ly.a) + row0 * ly.d_in, ly.d_in, valid, wave, lane);
  const f32x16 xg = gram_part<F16>(static_cast<const uint16_t*>(ly.g) + row0 * ly.d_out, ly.d_out, valid, wave, lane);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    part_a[wave][r][lane] = xa[r];
    part_g[wave][r][lane] = xg[r];
  }
  __syncthreads();
  // Register r of lane x holds row 8 (r >> 2) + 4 (x >> 5) + (r & 3), column x & 31; this thread: registers
  // wave and wave + 8.  Row sums inside the row's own sample, then the T rows of each sample.
  float row_sum[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = wave + 8 * h;
    float sa = 0.f, sg = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      sa += part_a[w][r][lane];
      sg += part_g[w][r][lane];
    }
    const int row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    float v = (lane & 31) / T == row / T ? sa * sg : 0.f;
#pragma unroll
    for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off);
    row_sum[h] = v;
  }
  __syncthreads();
  float* rows = &part_a[0][0][0];
  if ((lane & 31) == 0) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = wave + 8 * h;
      rows[8 * (r >> 2) + 4 * (lane >> 5) + (r & 3)] = row_sum[h];
    }
  }
  __syncthreads();
  if (tid >= begin && tid < end) {
    float s = 0.f;
    for (int t = 0; t < T; ++t) s += rows[tid * T + t];
    store_norm(ga, nc, l, i0 + tid, s, sqnorm);
  }
  finish_norms<kThreads>(ga, nc, sqnorm, reinterpret_cast<unsigned*>(rows));
}

// 33 to 64 tokens: a workgroup to a sample, its rows read once, the three 32 x 32 tiles on and above the diagonal side by
// side.  Norms, us, on the large-tile kernel (which pays for 128 rows) and here: 48 tokens, 7 samples of five layers 512 + 512
// 12.3, 7.6; 32 of twelve 768 + 2304 .. 3072 46.9, 28.2; 128 of sixteen 392 + 296 57.1, 46.5.  Like the form above it reads no more than
// some 28 GB/s a workgroup from memory (twice the loads in flight: the same), so samples of many values stay on large tiles: one
// of 64 tokens, 20 layers 1792 + 5376 .. 7168, a step 226 us there and 238 here; of 544 + 1632 .. 2176 57.7 and 51.0.
// Error against 64 bits: 0.6 to 1.1e-7 of the norm, there up to 2.2e-7.
constexpr int kPairDepth = kDepth / 2;           // of each half: kDepth loads in flight
template <bool F16>
__device__ __forceinline__ void gram_parts3(const uint16_t* x, int T, int width, int wave, int lane, f32x16 (&acc)[3]) {
#pragma unroll
  for (int n = 0; n < 3; ++n)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[n][r] = 0.f;
  const int t = lane & 31, u = kRows + t;
  const uint16_t* rt = x + (size_t)t * width;
  const uint16_t* ru = x + (size_t)min(u, T - 1) * width;
  for (int k0 = wave * 16; k0 < width; k0 += kPairDepth * kWaves * 16) {
    bf16x8 f[kPairDepth], h[kPairDepth];
#pragma unroll
    for (int q = 0; q < kPairDepth; ++q) {
      const int k = k0 + q * kWaves * 16 + 8 * (lane >> 5);
      uint4 w = make_uint4(0, 0, 0, 0), v = w;
      if (k < width) w = *reinterpret_cast<const uint4*>(rt + k);
      if (k < width && u < T) v = *reinterpret_cast<const uint4*>(ru + k);
      f[q] = __builtin_bit_cast(bf16x8, w);
      h[q] = __builtin_bit_cast(bf16x8, v);
    }
#pragma unroll
    for (int q = 0; q < kPairDepth; ++q) {
      acc[0] = mfma16<F16>(f[q], f[q], acc[0]);
      acc[1] = mfma16<F16>(f[q], h[q], acc[1]);
      acc[2] = mfma16<F16>(h[q], h[q], acc[2]);
    }
  }
}

template <bool F16>
__global__ void __launch_bounds__(kThreads, 4)
ghost_pair_kernel(const GroupArgs ga, float* sqnorm, const NormClip nc, int first) {
  // 64 KiB and 128 registers: two workgroups per compute unit (48 tokens, 2048 samples of two layers 392 + 296: 88 us with 142
  // registers and one, 60 so; 24 + 16 57, 37, and without the sums of waves that had no columns 28)
  __shared__ float part_a[kWaves][16][64], part_g[kWaves][16][64];
  __shared__ float wave_sum[kWaves];
  const int block = first + blockIdx.x;
  const int l = layer_of(ga, block);
  const GroupLayer& ly = ga.layer[l];
  const int T = ly.T, i = block - ly.tile_begin;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t row0 = (size_t)i * T;
  const int used = min(kWaves, (max(ly.d_in, ly.d_out) + 15) / 16);        // the other waves' sums are zeros: they stay out
  f32x16 xa[3], xg[3];
  gram_parts3<F16>(static_cast<const uint16_t*>(ly.a) + row0 * ly.d_in, T, ly.d_in, wave, lane, xa);
  if (wave < used)
#pragma unroll
    for (int r = 0; r < 16; ++r) part_a[wave][r][lane] = xa[0][r];       // at once: 16 registers that the g side can use
  gram_parts3<F16>(static_cast<const uint16_t*>(ly.g) + row0 * ly.d_out, T, ly.d_out, wave, lane, xg);
  float sum = 0.f;
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    if (n > 0) __syncthreads();                        // the last tile's parts are read
    if (wave < used)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (n > 0) part_a[wave][r][lane] = xa[n][r];
        part_g[wave][r][lane] = xg[n][r];
      }
    __syncthreads();
    // This thread: registers wave and wave + 8 of lane `lane` of every wave; row 8 (r >> 2) + 4 (lane >> 5) + (r & 3) of one
    // half, column lane & 31 of the other.  Rows past the sample are zeros, beside an infinity NaN: they stay out.
    float s = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = wave + 8 * h;
      float sa = 0.f, sg = 0.f;
      if (used == kWaves) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
          sa += part_a[w][r][lane];
          sg += part_g[w][r][lane];
        }
      } else {
        for (int w = 0; w < used; ++w) {
          sa += part_a[w][r][lane];
          sg += part_g[w][r][lane];
        }
      }
      const int row = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3), col = lane & 31;
      const bool in = n == 0 || kRows + (n == 1 ? col : max(row, col)) < T;
      s = in ? fmaf(sa, sg, s) : s;
    }
    sum += n == 1 ? 2.f * s : s;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) wave_sum[wave] = sum;
  __syncthreads();
  if (tid == 0) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += wave_sum[w];
    store_norm(ga, nc, l, i, s, sqnorm);
  }
  finish_norms<kThreads>(ga, nc, sqnorm, reinterpret_cast<unsigned*>(&part_a[0][0][0]));
}

}  // namespace

bool ghost_pair_supports(int T, int d, int p) {
  constexpr int64_t kMostValues = 300000;
  return T > kRows && T <= 2 * kRows && T * ((int64_t)d + p) <= kMostValues;
}

// Large samples, many rounds of them: one workgroup to a compute unit, by LDS that it does not use.  64 tokens, 2048 + 1024: 2048
// samples 186 us so and 197 with two, 6000 527 and 566, but 600 52 and 46; of 760 + 520, 6000 509 and 502.
constexpr int kWideValues = 128 * 1024, kWideSamples = 1024, kSoleLds = 32 * 1024;

template <bool F16>
dp_status launch_pair_t(const GroupArgs& ga, float* sqnorm, const NormClip& nc, hipStream_t s) {
  int lds = 0;
  if (ga.total_blocks >= kWideSamples)
    for (int l = 0; l < ga.n_layers; ++l)
      if ((int64_t)ga.layer[l].T * ((int64_t)ga.layer[l].d_in + ga.layer[l].d_out) > kWideValues) lds = kSoleLds;
  if (lds > 0) {
    static ReadyTable ready;
    dp_status st = allow_big_lds(ghost_pair_kernel<F16>, lds, ready);
    if (st != DP_OK) return st;
  }
  return launch_in_runs(ga.total_blocks, [&](dim3 grid, int first) {
    hipLaunchKernelGGL(ghost_pair_kernel<F16>, grid, dim3(kThreads), lds, s, ga, sqnorm, nc, first);
  });
}

dp_status launch_ghost_pair_group(const GroupArgs& ga, float* sqnorm, const NormClip& nc, hipStream_t s) {
  return ga.f16 ? launch_pair_t<true>(ga, sqnorm, nc, s) : launch_pair_t<false>(ga, sqnorm, nc, s);
}

bool ghost_brief_supports(int T) { return T <= kRows; }

// Workgroups of a layer, each with one of `parts` shares of the samples that fit the rows.  (A share may be empty: of the last rows.)
int64_t ghost_brief_blocks(int B, int T, int parts) {
  const int per = kRows / T;
  return (int64_t)((B + per - 1) / per) * parts;
}

int ghost_brief_max_parts(int B, int T) { return std::min(kRows / T, B); }

dp_status launch_ghost_brief_group(const GroupArgs& ga, float* sqnorm, const NormClip& nc, hipStream_t s) {
  return launch_in_runs(ga.total_blocks, [&](dim3 grid, int first) {
    if (ga.f16)
      hipLaunchKernelGGL(ghost_brief_kernel<true>, grid, dim3(kThreads), 0, s, ga, sqnorm, nc, first);
    else
      hipLaunchKernelGGL(ghost_brief_kernel<false>, grid, dim3(kThreads), 0, s, ga, sqnorm, nc, first);
  });
}

}  // namespace dpbk
