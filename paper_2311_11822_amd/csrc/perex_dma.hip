// Instantiated per-sample norm on the matrix cores (appendix A.1 of the
// paper, left side of eq. "mixed ghost norm"):  sqnorm[i] = || a_i^T g_i ||_F^2.
//
// One workgroup owns (sample, tile of the d_in x d_out gradient): it contracts over the
// sample's T token rows (tn_pipeline.h), squares and adds, and, on request, keeps the tile of G_i (appendix A.2
// applied to this path).
#include <type_traits>

#include "dp_internal.h"
#include "tile_order.h"
#include "tn_pipeline.h"

namespace dpbk {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4v;

template <class S, bool F16>
__global__ void __launch_bounds__(S::NT, S::NT == 256 ? 2 : 1)
perex_dma_kernel(const GroupArgs ga, float* __restrict__ partials) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];

  // The tiles of one (layer, sample) read the same panels of a_i and g_i: numbered consecutively
  // and dealt to the XCDs in contiguous eighths, they meet in one L2.
  const int item = contiguous_eighth(blockIdx.x, ga.total_blocks);
  const int l = layer_of(ga, item);
  const GroupLayer& ly = ga.layer[l];
  const int local = item - ly.tile_begin;
  const int sample = local / ly.tiles_per_sample;
  const int tile = local - sample * ly.tiles_per_sample;
  const int d = ly.d_in, p = ly.d_out;
  const int tiles_n = (p + S::BN - 1) / S::BN;
  const int m0 = (tile / tiles_n) * S::BM, n0 = (tile % tiles_n) * S::BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = (wave / S::WN) * S::WTM, wn = (wave % S::WN) * S::WTN;

  f32x16 acc[S::TM][S::TN];
  tn_contract<S, F16, false>(ly.a, ly.g, ly.T, d, p, sample, ga.B, nullptr, 0.f, m0, n0,
                             (unsigned)(uintptr_t)lds_raw, acc);
  __syncthreads();                                      // LDS is reused below

  // The MFMAs take the g fragment as first operand and the a fragment as second, so a wave holds
  // the transposed product: lane l has gradient row (l & 31) of a 32 x 32 tile and the columns
  // 8 q + 4 (l >> 5) + e (q, e = 0 .. 3) in register 4 q + e.
  if (ly.out) {
    float* dst = ly.out + (size_t)sample * d * p;
#pragma unroll
    for (int x = 0; x < S::TM; ++x)
#pragma unroll
      for (int y = 0; y < S::TN; ++y) {
        const int row = m0 + wm + x * 32 + (lane & 31);
        const int col0 = n0 + wn + y * 32 + 4 * (lane >> 5);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (row < d && col0 + 8 * q < p) {
            const f32x4v w = {acc[x][y][4 * q], acc[x][y][4 * q + 1], acc[x][y][4 * q + 2], acc[x][y][4 * q + 3]};
            *reinterpret_cast<f32x4v*>(dst + (size_t)row * p + col0 + 8 * q) = w;
          }
      }
  }

  // One partial sum per 128 x 128, added in the same order on either tile (four 64 x 64 pieces, two MFMA rows each):
  // the tile is chosen by what else is in the launch, and a layer's norm must not depend on that.
  constexpr int SIDE = S::BM / 128, SUBS = SIDE * SIDE, PIECES = S::TM / 2;
  float* red = reinterpret_cast<float*>(lds_raw);
  float sum[PIECES];
#pragma unroll
  for (int h = 0; h < PIECES; ++h) sum[h] = 0.f;
  if (m0 + wm + S::WTM <= d && n0 + wn + S::WTN <= p) {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < S::TN; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int h = 0; h < PIECES; ++h) sum[h] = fmaf(acc[2 * h + x][y][r], acc[2 * h + x][y][r], sum[h]);
  } else {
    // Rows and columns past the layer's edge were loaded as zeros, but an infinity of the other operand
    // makes NaN of them: they stay out.  d_out is a multiple of 8: eight columns, four to a half wave, are in or out.
#pragma unroll
    for (int x = 0; x < S::TM; ++x)
      if (m0 + wm + x * 32 + (lane & 31) < d)
#pragma unroll
        for (int y = 0; y < S::TN; ++y)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (n0 + wn + y * 32 + 8 * q < p)
#pragma unroll
              for (int r = 4 * q; r < 4 * q + 4; ++r) sum[x / 2] = fmaf(acc[x][y][r], acc[x][y][r], sum[x / 2]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
#pragma unroll
    for (int h = 0; h < PIECES; ++h) sum[h] += __shfl_xor(sum[h], off);
#pragma unroll
  for (int h = 0; h < PIECES; ++h) {
    const int row = wm + 64 * h;                        // of the piece, inside the tile
    if (lane == 0) red[4 * (row / 128 * SIDE + wn / 128) + 2 * (row / 64 % 2) + wn / 64 % 2] = sum[h];
  }
  __syncthreads();
  if (threadIdx.x < SUBS) {
    float total = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) total += red[4 * threadIdx.x + w];
    const int row = m0 + 128 * (threadIdx.x / SIDE), col = n0 + 128 * (threadIdx.x % SIDE);
    const int subs_m = (d + 127) / 128, subs_n = (p + 127) / 128;
    if (row < d && col < p)
      partials[ly.part_begin + (sample * subs_m + row / 128) * subs_n + col / 128] = total;
  }
}

template <class S, bool F16>
dp_status launch_perex_dma_t(const GroupArgs& ga, float* partials, hipStream_t s) {
  auto kernel = perex_dma_kernel<S, F16>;
  static ReadyTable ready;
  dp_status st = allow_big_lds(kernel, S::LDS_BYTES, ready);
  if (st != DP_OK) return st;
  hipLaunchKernelGGL(kernel, dim3(ga.total_blocks), dim3(S::NT), S::LDS_BYTES, s, ga, partials);
  return hip_status(hipGetLastError());
}

}  // namespace

// 32-bit byte offsets inside a sample's slab, bit 31 as the "fetch zeros" marker, and the
// prefetch runs up to NSTAGE blocks past the last token row without wrapping.
bool perex_dma_supports(int T, int d, int p) {
  const int64_t rows = (int64_t)T + (MidTile::NSTAGE + 1) * MidTile::BK;
  return rows * d * 2 < (int64_t)1 << 31 && rows * p * 2 < (int64_t)1 << 31;
}

// big: ga's tiles are 256 x 256 instead of 128 x 128.
dp_status launch_perex_dma_group(const GroupArgs& ga, float* partials, bool big, hipStream_t s) {
  if (big) return ga.f16 ? launch_perex_dma_t<BigTile, true>(ga, partials, s) : launch_perex_dma_t<BigTile, false>(ga, partials, s);
  return ga.f16 ? launch_perex_dma_t<MidTile, true>(ga, partials, s) : launch_perex_dma_t<MidTile, false>(ga, partials, s);
}

}  // namespace dpbk
