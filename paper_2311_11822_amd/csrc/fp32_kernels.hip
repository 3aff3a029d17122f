// fp32-input forms of the three contractions, grouped over layers: one launch for the norms of a
// stack and one for its gradients (+ noise).  fp32 layers are small (a few thousand weights), so
// what bounds them is latency: launches, and the serial chain of a workgroup.  Products run on the
// fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands and sums, 64 clocks for 32 x 32 x 2), whose
// operands come straight from global memory: one register per lane holds 32 consecutive columns
// of two token rows (TN products), or a quarter of a float4 of 32 token rows (NT products), so no LDS
// staging and no barrier sits in the loops.  The eight waves of a workgroup split the contraction (or
// the tiles) and meet once, in LDS, in a fixed order: no atomics, the same bits every time.
// Measured on eight layers of width 64..256 (B = 16, T = 48): one thread per output and one launch per
// layer took 2904 us a step (182 us per gradient, 174 us per norm); this form 29 us: norms, clip factors, gradients.
#include <algorithm>

#include "clip.h"
#include "dp_internal.h"

namespace dpbk {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4v;
constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kTile = 32;                        // output tile edge = MFMA edge
constexpr int kChunk = 16;                       // token rows per work item: 8 MFMAs

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

// Sum over the workgroup in a fixed order; every thread calls it, the result is valid in thread 0.
__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();                               // earlier readers of `red` are done
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) s += red[w];
  return s;
}

// Four consecutive elements k .. k + 3 of a row of `width`, zeros past its end.  VEC: width is a
// multiple of 4 (rows are then 16-byte aligned).
template <bool VEC>
__device__ __forceinline__ f32x4v load4(const float* row, int k, int width) {
  f32x4v v = {0.f, 0.f, 0.f, 0.f};
  if constexpr (VEC) {
    if (k < width) v = *reinterpret_cast<const f32x4v*>(row + k);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < width) v[e] = row[k + e];
  }
  return v;
}

// This wave's part of the 32 x 32 tile (t0, u0) of x x^T: the k's of every kWaves-th group of 8.
// The order of the k's inside an MFMA is free as long as both operands share it.
template <bool VEC>
__device__ __forceinline__ f32x16 gram_part(const float* x, int T, int width, int t0, int u0, int wave, int lane) {
  f32x16 acc = zero16();
  const bool same = t0 == u0;
  const int t = t0 + (lane & 31), u = u0 + (lane & 31);
  const float* rt = x + (size_t)min(t, T - 1) * width;
  const float* ru = x + (size_t)min(u, T - 1) * width;
  const int wt = t < T ? width : 0, wu = u < T ? width : 0;          // rows past the sample: zeros
  for (int k0 = wave * 8; k0 < width; k0 += 4 * kWaves * 8) {
    f32x4v a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + q * kWaves * 8 + 4 * (lane >> 5);
      a[q] = load4<VEC>(rt, k, wt);
      b[q] = same ? a[q] : load4<VEC>(ru, k, wu);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      // past the width there are zeros only (widths of single loads: the branch costs their order more than it saves)
      if (!VEC || k0 + q * kWaves * 8 < width) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = mfma32(a[q][e], b[q][e], acc);
      }
  }
  return acc;
}

// The same of the tiles (0, 0), (0, 32), (32, 32) of a sample of 33 to 64 tokens: its rows read once, no load waits for
// another tile's sums.  Widths that are multiples of 4: eight layers of width 64 .. 256, 16 x 48 tokens, 15.4 -> 10.4 us; of others,
// with their single loads, slower (ten to 40 wide, 28 x 56: 11.0 -> 17.4).
__device__ __forceinline__ void gram_parts3(const float* x, int T, int width, int wave, int lane, f32x16 (&acc)[3]) {
#pragma unroll
  for (int n = 0; n < 3; ++n) acc[n] = zero16();
  const int t = lane & 31, u = 32 + (lane & 31);
  const float* rt = x + (size_t)t * width;
  const float* ru = x + (size_t)min(u, T - 1) * width;
  const int wu = u < T ? width : 0;
  for (int k0 = wave * 8; k0 < width; k0 += 4 * kWaves * 8) {
    f32x4v a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int k = k0 + q * kWaves * 8 + 4 * (lane >> 5);
      a[q] = load4<true>(rt, k, width);
      b[q] = load4<true>(ru, k, wu);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (k0 + q * kWaves * 8 < width) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc[0] = mfma32(a[q][e], a[q][e], acc[0]);
          acc[1] = mfma32(a[q][e], b[q][e], acc[1]);
          acc[2] = mfma32(b[q][e], b[q][e], acc[2]);
        }
      }
  }
}

__device__ __forceinline__ f32x16 gram_part(const float* x, int T, int width, int t0, int u0, int wave, int lane) {
  return (width & 3) ? gram_part<false>(x, T, width, t0, u0, wave, lane)
                     : gram_part<true>(x, T, width, t0, u0, wave, lane);
}

// Operands of one work item of a TN product: rows [t0, t0 + kChunk) of a and g (already offset to
// the sample), columns j of a and k of g per lane; two rows per register, zeros outside.
struct TnItem {
  float a[kChunk / 2], g[kChunk / 2];
};
__device__ __forceinline__ void load_item(TnItem& it, const float* a, const float* g, int t0, int T, int d, int p,
                                          int j, int k, int lane) {
#pragma unroll
  for (int q = 0; q < kChunk / 2; ++q) {
    const int t = t0 + 2 * q + (lane >> 5);
    it.a[q] = t < T && j < d ? a[(size_t)t * d + j] : 0.f;
    it.g[q] = t < T && k < p ? g[(size_t)t * p + k] : 0.f;
  }
}
// The same through buffer descriptors over the sample's rows, whose range check makes the zeros: no masks around the loads.
// ja, kg: byte of the lane's column in a row, or kOutside.
constexpr unsigned kOutside = 0x80000000u;
__device__ __forceinline__ void load_item(TnItem& it, __amdgpu_buffer_rsrc_t a, __amdgpu_buffer_rsrc_t g, int t0, int d, int p,
                                          unsigned ja, unsigned kg, int lane) {
#pragma unroll
  for (int q = 0; q < kChunk / 2; ++q) {
    const unsigned t = t0 + 2 * q + (lane >> 5);
    it.a[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(a, t * d * 4u + ja, 0, 0));
    it.g[q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(g, t * p * 4u + kg, 0, 0));
  }
}
// The g operand first: lane l then holds row l & 31 of the tile and runs of four consecutive
// columns, 8 q + 4 (l >> 5) + e in register 4 q + e.
__device__ __forceinline__ f32x16 mul_item(const TnItem& it, f32x16 acc) {
#pragma unroll
  for (int q = 0; q < kChunk / 2; ++q) acc = mfma32(it.g[q], it.a[q], acc);
  return acc;
}

// Squared per-sample norms, one workgroup per (layer, sample), by the layer's path (appendix A.1):
// ghost: sum over token pairs of (a_t . a_u)(g_t . g_u), tile pairs on and above the diagonal;
// instantiated: || a_i^T g_i ||_F^2.
// A tile's entries outside the layer (past d, p or T) are selected out before they are added: their
// zero operands meet the other side's values, and an infinity there would make them NaN.
// VEC: every width of the launch is a multiple of 4, every slab small (small_slabs).  (A kernel of its own: beside the single loads of other widths the
// compiler orders either form's loads worse; eight layers ten to 40 wide, 28 x 56 tokens, 34.8 us a step apart, 36.6 to 45.8
// in one.)
// Two workgroups to a compute unit, which 128 registers allow (the three tiles side by side took 145 of them, and one workgroup was alone):
// 4096 samples, one and two to a unit: 16 tokens, two layers 256 + 256 190, 130 us; 48, two of 64 + 128 208, 148; instantiated,
// 8, two of 64 x 64 47, 30.
template <bool VEC>
__global__ void __launch_bounds__(kThreads, 4)
norms_f32_kernel(const GroupArgs ga, float* sqnorm, const NormClip nc, int first) {
  __shared__ float part_a[kWaves][16][64], part_g[kWaves][16][64];   // 64 KiB
  const unsigned block = first + blockIdx.x;
  const int l = block / ga.B, i = block - l * ga.B;
  const GroupLayer& ly = ga.layer[l];
  const int T = ly.T, d = ly.d_in, p = ly.d_out;
  const float* a = static_cast<const float*>(ly.a) + (size_t)i * T * d;
  const float* g = static_cast<const float*>(ly.g) + (size_t)i * T * p;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float sum = 0.f;
  auto put = [&](float (*part)[16][64], const f32x16& acc) {
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][r][lane] = acc[r];
  };
  auto total = [&](float (*part)[16][64], int e) {      // element e of the tile over the waves
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s += part[w][e >> 6][e & 63];
    return s;
  };

  // Register r of a lane: place run(r) along the tile's Gram rows (gradient columns), lane & 31 along the other side.
  auto run = [&](int r) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); };

  if (ly.path == DP_PATH_GHOST) {
    auto add_parts = [&](int t0, int u0) {                 // the tile whose parts are in LDS
      __syncthreads();
      float s = 0.f;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float va = total(part_a, tid + h * kThreads), vg = total(part_g, tid + h * kThreads);
        const bool in = t0 + run(wave + h * kWaves) < T && u0 + (lane & 31) < T;
        s = in ? fmaf(va, vg, s) : s;
      }
      sum += t0 == u0 ? s : 2.f * s;
      __syncthreads();
    };
    auto add_tile = [&](int t0, int u0, const f32x16& xa, const f32x16& xg) {
      put(part_a, xa);
      put(part_g, xg);
      add_parts(t0, u0);
    };
    if (VEC && T > kTile && T <= 2 * kTile) {
      f32x16 xa[3], xg[3];
      gram_parts3(a, T, d, wave, lane, xa);
      put(part_a, xa[0]);                                  // at once: 16 registers that the g side can use
      gram_parts3(g, T, p, wave, lane, xg);
      put(part_g, xg[0]);
      add_parts(0, 0);
      add_tile(0, kTile, xa[1], xg[1]);
      add_tile(kTile, kTile, xa[2], xg[2]);
    } else {
      for (int t0 = 0; t0 < T; t0 += kTile)
        for (int u0 = t0; u0 < T; u0 += kTile)
          if constexpr (VEC)
            add_tile(t0, u0, gram_part<true>(a, T, d, t0, u0, wave, lane), gram_part<true>(g, T, p, t0, u0, wave, lane));
          else
            add_tile(t0, u0, gram_part(a, T, d, t0, u0, wave, lane), gram_part(g, T, p, t0, u0, wave, lane));
    }
  } else {
    const int tn = (p + kTile - 1) / kTile, tiles = ((d + kTile - 1) / kTile) * tn;
    const int items = (T + kChunk - 1) / kChunk;
    // The waves share the tokens of each tile where that employs more of them than a tile to each (5 x 176, 7 tokens, 406
    // samples of 11 layers: 59 us before there were tiles, 77 shared, 29 so).
    const bool split = tiles < kWaves && items > tiles;
    const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)a, 0, T * d * 4, 0x00020000);
    const auto rg = __builtin_amdgcn_make_buffer_rsrc((void*)g, 0, T * p * 4, 0x00020000);
    for (int tile = split ? 0 : wave; tile < tiles; tile += split ? 1 : kWaves) {
      const int n0 = (tile % tn) * kTile;
      const int j = (tile / tn) * kTile + (lane & 31), k = n0 + (lane & 31);
      f32x16 acc = zero16();
      for (int c = split ? wave : 0; c < items; c += split ? kWaves : 1) {
        TnItem it;
        if constexpr (VEC)
          load_item(it, ra, rg, c * kChunk, d, p, j < d ? 4u * j : kOutside, k < p ? 4u * k : kOutside, lane);
        else
          load_item(it, a, g, c * kChunk, T, d, p, j, k, lane);
        acc = mul_item(it, acc);
      }
      // Columns of a and g left in the tile, formed anew: from j < d the compiler makes a mask that it holds through the
      // loads above, and waits for each of those in turn (300 tokens, 11 x 216: 30 -> 65 us).
      int left_d = d - (tile / tn) * kTile, left_p = p - n0;
      asm volatile("" : "+s"(left_d), "+s"(left_p));
      const bool in_d = (lane & 31) < left_d, whole = left_d >= kTile && left_p >= kTile;
      if (split) {
        put(part_a, acc);
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const float v = total(part_a, tid + h * kThreads);
          const float in = in_d && run(wave + h * kWaves) < left_p ? v : 0.f;
          sum = fmaf(in, in, sum);
        }
        __syncthreads();
      } else if (whole) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sum = fmaf(acc[r], acc[r], sum);
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float in = in_d && run(r) < left_p ? acc[r] : 0.f;
          sum = fmaf(in, in, sum);
        }
      }
    }
  }
  const float s = block_sum(sum, &part_g[0][0][0]);
  if (tid == 0) store_norm(ga, nc, l, i, s, sqnorm);
  finish_norms<kThreads>(ga, nc, sqnorm, reinterpret_cast<unsigned*>(&part_a[0][0][0]));
}

// Clip-weighted gradient (section 3): grad[j,k] = sum_i C_i sum_t a[i,t,j] g[i,t,k] (+ noise, eq. (1)).
// One workgroup per 32 x 32 tile; its waves take contiguous runs of the (sample, 16 tokens) items.
// An item's product is formed unweighted and folded in as total += C_i * item; a sample with
// C_i == 0 does not enter.
// SMALL: every sample's a and g are less than 2 GiB, so that they load through buffer descriptors (samples that do not
// enter too: the loads do not wait for the weight).
template <bool SMALL>
__global__ void __launch_bounds__(kThreads)
clipped_grad_f32_kernel(const GroupArgs ga, const float* __restrict__ C_all, const NoiseArgs na, int first) {
  __shared__ float part[kWaves][16][64];                 // 32 KiB
  const int block = first + blockIdx.x;
  const int l = layer_of(ga, block);
  const GroupLayer& ly = ga.layer[l];
  const int T = ly.T, d = ly.d_in, p = ly.d_out;
  const int tile = block - ly.tile_begin, tn = (p + kTile - 1) / kTile;
  const int m0 = (tile / tn) * kTile, n0 = (tile % tn) * kTile;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const float* a = static_cast<const float*>(ly.a);
  const float* g = static_cast<const float*>(ly.g);
  const float* __restrict__ C = C_all + ly.c_off;
  const int j = m0 + (lane & 31), k = n0 + (lane & 31);

  const int per_sample = (T + kChunk - 1) / kChunk;
  const int64_t items = (int64_t)ga.B * per_sample;
  const int64_t begin = items * wave / kWaves, end = items * (wave + 1) / kWaves;
  int i = (int)(begin / per_sample), c = (int)(begin - (int64_t)i * per_sample);
  f32x16 sum = zero16();
  TnItem cur, next;
  float wc = 0.f, wn = 0.f;
  auto fetch = [&](TnItem& it, float& w) {               // item (i, c), then step to the next one
    w = C[i];
    if constexpr (SMALL) {                               // whether it counts or not: the loads need not wait for the weight
      const auto ra = __builtin_amdgcn_make_buffer_rsrc((void*)(a + (size_t)i * T * d), 0, T * d * 4, 0x00020000);
      const auto rg = __builtin_amdgcn_make_buffer_rsrc((void*)(g + (size_t)i * T * p), 0, T * p * 4, 0x00020000);
      load_item(it, ra, rg, c * kChunk, d, p, j < d ? 4u * j : kOutside, k < p ? 4u * k : kOutside, lane);
    } else if (w != 0.f) {
      load_item(it, a + (size_t)i * T * d, g + (size_t)i * T * p, c * kChunk, T, d, p, j, k, lane);
    }
    if (++c == per_sample) {
      c = 0;
      ++i;
    }
  };
  if (begin < end) fetch(cur, wc);
  for (int64_t n = begin; n < end; ++n) {
    if (n + 1 < end) fetch(next, wn);
    if (wc != 0.f) {
      const f32x16 acc = mul_item(cur, zero16());
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[r] = fmaf(wc, acc[r], sum[r]);
    }
    cur = next;
    wc = wn;
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) part[wave][r][lane] = sum[r];
  __syncthreads();
  if (tid >= 256) return;
  // thread: one run of four consecutive columns (register group q of lane `lane`)
  const int q = tid >> 6;
  const int row = m0 + (lane & 31), col = n0 + 8 * q + 4 * (lane >> 5);
  if (row >= d || col >= p) return;
  const int n = min(4, p - col);
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) v[e] += part[w][4 * q + e][lane];
  }
  float* out = ly.out + (size_t)row * p + col;
  if (ga.accumulate) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) v[e] = out[e] + v[e];
  }
  if (na.stddev != 0.f) {
    const uint64_t idx = na.layer_off[l] + (uint64_t)row * p + col;
    if (idx + n > na.lo && idx < na.hi) {
      if ((idx & 3) == 0) {
        float z[4];
        normal_block(idx >> 2, na.step_lo, na.step_hi, na.rk, z);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (idx + e >= na.lo && idx + e < na.hi) v[e] = fmaf(na.stddev, z[e], v[e]);
      } else {                                           // the run straddles generator blocks
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (idx + e >= na.lo && idx + e < na.hi) {
            float z[4];
            normal_block((idx + e) >> 2, na.step_lo, na.step_hi, na.rk, z);
            const int s = (int)((idx + e) & 3);
            v[e] = fmaf(na.stddev, s == 0 ? z[0] : s == 1 ? z[1] : s == 2 ? z[2] : z[3], v[e]);
          }
      }
    }
  }
  if ((p & 3) == 0) {
    *reinterpret_cast<f32x4v*>(out) = f32x4v{v[0], v[1], v[2], v[3]};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < n) out[e] = v[e];
  }
}

// Byte offsets inside a sample stay below kOutside, those of the last chunk's rows past the end included.
bool small_slabs(const GroupLayer& ly) {
  return ((int64_t)ly.T + kChunk) * std::max(ly.d_in, ly.d_out) * 4 < (int64_t)1 << 31;
}

}  // namespace

int64_t clipped_grad_f32_tiles(int d, int p) {
  return (((int64_t)d + kTile - 1) / kTile) * (((int64_t)p + kTile - 1) / kTile);
}

dp_status launch_norms_f32_group(const GroupArgs& ga, float* sqnorm, const NormClip& nc, hipStream_t s) {
  bool vec = true;
  for (int l = 0; l < ga.n_layers; ++l) vec = vec && ((ga.layer[l].d_in | ga.layer[l].d_out) & 3) == 0 && small_slabs(ga.layer[l]);
  auto kernel = vec ? norms_f32_kernel<true> : norms_f32_kernel<false>;
  return launch_in_runs(ga.total_blocks, [&](dim3 grid, int first) {
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, ga, sqnorm, nc, first);
  });
}

dp_status launch_clipped_grad_f32_group(const GroupArgs& ga, const float* C, const NoiseArgs& na, hipStream_t s) {
  bool small = true;
  for (int l = 0; l < ga.n_layers; ++l) small = small && small_slabs(ga.layer[l]);
  auto kernel = small ? clipped_grad_f32_kernel<true> : clipped_grad_f32_kernel<false>;
  return launch_in_runs(ga.total_blocks, [&](dim3 grid, int first) {
    hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, ga, C, na, first);
  });
}

}  // namespace dpbk
