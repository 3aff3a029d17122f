// Layer-wise clipping in one pass over a layer's a and g (section 3.3 (II) of the paper and the
// formula of its appendix on the hook-free implementation): with one clipping group per layer
// the factor C_{l,i} depends on layer l alone, so for a layer whose whole d_in x d_out gradient
// fits one workgroup tile the same kernel can instantiate G_i = a_i^T g_i (appendix A.1, left
// side of eq. "mixed ghost norm"), take its norm, turn it into C_i (section 2.1) and add
// C_i G_i to the running sum (section 3, "DP gradient") -- nothing is book-kept and a, g are read
// once.
//
// One workgroup owns (layer, chunk of consecutive samples).  Per sample it runs the token
// contraction of the instantiated-norm kernel (tn_tile.h machinery) into one accumulator set,
// reduces the sum of squares over the workgroup in a fixed order, and adds C_i times the
// accumulators to a second set.  The norm is added up in the order of the kernel that takes the layer elsewhere, the same bits:
// which of the two forms a layer takes is a matter of its stack, its norm and factor are not.  The chunk's weighted sum goes to a workspace; a second small
// kernel adds the chunks in order, adds the noise of eq. (1) and writes the gradient.  No
// atomics: the result is deterministic.
#include <type_traits>

#include "clip.h"
#include "dp_internal.h"
#include "tn_tile.h"

namespace dpbk {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4v;

struct FusedArgs {
  int mode;
  float stability;
  float R[kMaxGroup];            // threshold of each layer of the launch
};

// One step of two butterfly sums at once: that of x stays in the lanes without bit OFF, that of y in those with it.
template <int OFF>
__device__ __forceinline__ float halves_sum(float x, float y, int lane) {
  const bool upper = lane & OFF;
  return (upper ? y : x) + __shfl_xor(upper ? x : y, OFF);
}

// GroupLayer fields as used here: tile_begin = first workgroup of the layer, tiles_per_sample =
// number of sample chunks, part_begin = float offset of the layer's [chunks][d_in * d_out]
// partial sums in the workspace, sq_index = row of sqnorm / C.
template <class S, bool F16>
__global__ void __launch_bounds__(S::NT, 2 * S::LDS_BYTES <= 163840 ? 2 : 1)
layerwise_fused_kernel(const GroupArgs ga, const FusedArgs fa, float* __restrict__ partial,
                       float* __restrict__ sqnorm, float* __restrict__ C_out) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  const int l = layer_of(ga, blockIdx.x);
  const GroupLayer& ly = ga.layer[l];
  const int chunk = blockIdx.x - ly.tile_begin;
  const int per = (ga.B + ly.tiles_per_sample - 1) / ly.tiles_per_sample;
  const int i0 = chunk * per, i1 = min(ga.B, i0 + per);

  TnTile<S> t;
  t.a = static_cast<const uint16_t*>(ly.a);
  t.g = static_cast<const uint16_t*>(ly.g);
  t.T = ly.T;
  t.d = ly.d_in;
  t.p = ly.d_out;
  t.m0 = 0;
  t.n0 = 0;
  const int nkb = (ly.T + S::BK - 1) / S::BK;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = (wave / S::WN) * S::WTM, wn = (wave % S::WN) * S::WTN;
  const int row0 = wm + (lane & 31), col0 = wn + 4 * (lane >> 5);       // the lane's first element
  // How the sums of squares of the 32 x 32 tiles go together: a 128 x 128 tile of perex_dma.hip wave by wave (kTile); the
  // four waves of perex_narrow.hip with 32 rows (kStrips), 32 columns (kFlat) or 32 x 64 each (kHalves); its tiles of 128 rows
  // or columns, one to a wave here (kTiles).
  enum { kTile, kStrips, kFlat, kHalves, kTiles };
  constexpr bool kSquare = S::TM == 2 && S::TN == 2 && S::WM == 2;
  static_assert(kSquare || (S::TM * S::TN == 4 && S::WM * S::WN == 4 && (S::WTM == 128 || S::WTN == 128)), "order of sums");
  const int order = !kSquare                                             ? kTiles
                    : ly.d_in > 64 && ly.d_out > 64                      ? kTile
                    : ly.d_out <= 32 || (ly.d_in > 32 && ly.d_out <= 64) ? kStrips
                    : ly.d_in <= 32                                      ? kFlat
                                                                         : kHalves;
  float* red = reinterpret_cast<float*>(lds);

  f32x16 total[S::TM][S::TN];
  zero_acc<S>(total);
  for (int i = i0; i < i1; ++i) {
    f32x16 acc[S::TM][S::TN];
    zero_acc<S>(acc);
    t.gload(i, 0);
    t.lds_store(lds);
    __syncthreads();
    for (int kb = 0, stage = 0; kb < nkb; ++kb, stage ^= 1) {
      const bool more = kb + 1 < nkb;
      if (more) t.gload(i, kb + 1);
      t.template compute<F16, true>(lds + stage * S::STAGE, acc);
      if (more) t.lds_store(lds + (stage ^ 1) * S::STAGE);
      __syncthreads();
    }
    // ||G_i||_F^2.  Rows and columns past the layer's edge were loaded as zeros and add nothing, unless an infinity of the other
    // operand made NaN of them: then they are taken out and it is added up again.
    float sq;
    for (bool again = false;; again = true) {
      float part[4], s = 0.f;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        if (n == 0 || (n % S::TN == 0 ? order != kTile : order == kFlat || order == kTiles)) s = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) s = fmaf(acc[n / S::TN][n % S::TN][r], acc[n / S::TN][n % S::TN][r], s);
        part[n] = s;
      }
      if constexpr (kSquare) {
        const float first = part[order == kFlat ? 0 : 1], second = order == kFlat ? part[1] : part[3];
        float v = halves_sum<32>(first, second, lane);
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if ((lane & 31) == 0) red[2 * wave + (lane >> 5)] = v;        // every LDS read of the loop is behind a barrier
        __syncthreads();
        if (order == kTile)                        // same order in every thread
          sq = red[1] + red[3] + red[5] + red[7];
        else if (order == kStrips)
          sq = (red[0] + red[1]) + (red[4] + red[5]);
        else if (order == kFlat)
          sq = (red[0] + red[1]) + (red[2] + red[3]);
        else
          sq = (red[0] + red[2]) + (red[1] + red[3]);
      } else {
        float v = halves_sum<16>(halves_sum<32>(part[0], part[1], lane), halves_sum<32>(part[2], part[3], lane), lane);
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off);
        v += __shfl_xor(v, 32);
        v += __shfl_xor(v, 16);
        if (lane == 0) red[wave] = v;
        __syncthreads();
        sq = (red[0] + red[2]) + (red[1] + red[3]);
      }
      if (sq == sq || again) break;
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (row0 + n / S::TN * 32 >= ly.d_in || col0 + n % S::TN * 32 + 8 * (r >> 2) >= ly.d_out) acc[n / S::TN][n % S::TN][r] = 0.f;
      __syncthreads();                             // red is read
    }
    __syncthreads();                               // red is overwritten by the next sample's tiles
    const float c = clip_factor(norm_of(sq), fa.mode, fa.R[l], fa.stability);
    if (threadIdx.x == 0) {
      sqnorm[(size_t)ly.sq_index * ga.B + i] = sq;
      C_out[(size_t)ly.sq_index * ga.B + i] = c;
    }
    if (c != 0.f) {
#pragma unroll
      for (int im = 0; im < S::TM; ++im)
#pragma unroll
        for (int jn = 0; jn < S::TN; ++jn)
#pragma unroll
          for (int r = 0; r < 16; ++r) total[im][jn][r] = fmaf(c, acc[im][jn][r], total[im][jn][r]);
    }
  }

  // the chunk's weighted sum, [d_in, d_out] row-major
  float* out = partial + ly.part_begin + (size_t)chunk * ly.d_in * ly.d_out;
#pragma unroll
  for (int im = 0; im < S::TM; ++im)
#pragma unroll
    for (int jn = 0; jn < S::TN; ++jn)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = row0 + im * 32, col = col0 + jn * 32 + 8 * q;
        if (row < ly.d_in && col < ly.d_out)
          *reinterpret_cast<f32x4v*>(out + (size_t)row * ly.d_out + col) =
              f32x4v{total[im][jn][4 * q], total[im][jn][4 * q + 1], total[im][jn][4 * q + 2], total[im][jn][4 * q + 3]};
      }
}

// grad[e] (+)= sum over the layer's chunks, in chunk order, (+ noise of eq. (1) at the element's
// global index, the same values dp_add_noise draws).  blockIdx.y = layer of the launch.
__global__ void __launch_bounds__(256)
layerwise_reduce_kernel(const GroupArgs ga, const float* __restrict__ partial, const NoiseArgs na) {
  const GroupLayer& ly = ga.layer[blockIdx.y];
  const int n = ly.d_in * ly.d_out;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  const float* src = partial + ly.part_begin + e;
  float v = 0.f;
  for (int c0 = 0; c0 < ly.tiles_per_sample; c0 += 8) {          // eight chunks in flight, added in order
    float x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[q] = c0 + q < ly.tiles_per_sample ? src[(size_t)(c0 + q) * n] : 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) v += x[q];
  }
  if (ga.accumulate) v += ly.out[e];
  if (na.stddev != 0.f) {
    const uint64_t idx = na.layer_off[blockIdx.y] + (uint64_t)e;
    if (idx >= na.lo && idx < na.hi) {
      float z[4];
      normal_block(idx >> 2, na.step_lo, na.step_hi, na.rk, z);
      const int k = (int)(idx & 3);
      v = fmaf(na.stddev, k == 0 ? z[0] : k == 1 ? z[1] : k == 2 ? z[2] : z[3], v);
    }
  }
  ly.out[e] = v;
}

// One workgroup tile holds the whole layer: 128 x 128, or a strip 512 x 32 / 32 x 512 (the shapes of low-rank adapter
// factors).
using FusedSquare = TnShape<128, 128, 64, 2, 2>;
using FusedTall = TnShape<512, 32, 64, 4, 1>;
using FusedWide = TnShape<32, 512, 64, 1, 4>;

template <class S, bool F16>
dp_status launch_fused_t(const GroupArgs& ga, const FusedArgs& fa, float* partial, float* sqnorm, float* C_out,
                         hipStream_t s) {
  auto kernel = layerwise_fused_kernel<S, F16>;
  static ReadyTable ready;
  dp_status st = allow_big_lds(kernel, (int)S::LDS_BYTES, ready);
  if (st != DP_OK) return st;
  hipLaunchKernelGGL(kernel, dim3(ga.total_blocks), dim3(S::NT), S::LDS_BYTES, s, ga, fa, partial, sqnorm, C_out);
  return hip_status(hipGetLastError());
}

}  // namespace

int layerwise_fused_shape(int d, int p) {
  if (d <= 128 && p <= 128) return 0;
  if (d <= 512 && p <= 32) return 1;
  if (d <= 32 && p <= 512) return 2;
  return -1;
}

dp_status launch_layerwise_fused(int shape, const GroupArgs& ga, const float* R, int mode, float stability, float* partial,
                                 float* sqnorm, float* C_out, hipStream_t s) {
  FusedArgs fa;
  fa.mode = mode;
  fa.stability = stability;
  for (int j = 0; j < ga.n_layers; ++j) fa.R[j] = R[j];
  for (int j = ga.n_layers; j < kMaxGroup; ++j) fa.R[j] = 1.f;
  auto launch = [&](auto f16) {
    constexpr bool F16 = decltype(f16)::value;
    return shape == 0   ? launch_fused_t<FusedSquare, F16>(ga, fa, partial, sqnorm, C_out, s)
           : shape == 1 ? launch_fused_t<FusedTall, F16>(ga, fa, partial, sqnorm, C_out, s)
                        : launch_fused_t<FusedWide, F16>(ga, fa, partial, sqnorm, C_out, s);
  };
  return ga.f16 ? launch(std::true_type{}) : launch(std::false_type{});
}

dp_status launch_layerwise_reduce(const GroupArgs& ga, const float* partial, const NoiseArgs& na, hipStream_t s) {
  int widest = 0;
  for (int j = 0; j < ga.n_layers; ++j) widest = std::max(widest, ga.layer[j].d_in * ga.layer[j].d_out);
  hipLaunchKernelGGL(layerwise_reduce_kernel, dim3((widest + 255) / 256, ga.n_layers), dim3(256), 0, s, ga,
                     partial, na);
  return hip_status(hipGetLastError());
}

}  // namespace dpbk
