// Instantiated per-sample norm of narrow layers (appendix A.1 of the paper, left side of eq. "mixed ghost
// norm"), d_in or d_out up to 64 (low-rank adapter factors):   sqnorm[i] = || a_i^T g_i ||_F^2, G_i kept on request.
//
// What bounds these layers is the stream over the wide operand.  A 128 x 128 tile (perex_dma.hip) pads the
// narrow one to 128 columns: as many LDS bytes and matrix instructions again for zeros.  Here the tile covers just
// the narrow side, 32 or 64 wide; one workgroup per (sample, 128 columns of the wide side), four LDS stages of 32
// rows, 40 or 48 KiB, so that three or four workgroups share a compute unit and their loads overlap.
// Measured, 24 adapter pairs 768 x 16, 16 x 256 tokens: 68 us on 128 x 128 tiles, 50 here (308 MB of operands: 6.2 TB/s).
#include "dp_internal.h"
#include "row_tile.h"
#include "tile_order.h"

namespace dpbk {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4v;
constexpr int BK = 32, NSTAGE = 4, NT = 256;

template <int BM_, int BN_, int WM_, int WN_>
struct Shape {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int TN = BN / WN / 32;                       // 32 rows x 32 TN columns per wave
  static constexpr int A_BYTES = BK * BM * 2, STAGE_BYTES = A_BYTES + BK * BN * 2;
  static constexpr int LOADS = kRowLoads<BM> + kRowLoads<BN>;
  static_assert(BM / WM == 32 && WM * WN == 4, "shape");
};
using Tall = Shape<128, 32, 4, 1>;
using Tall2 = Shape<128, 64, 4, 1>;
using Flat = Shape<32, 128, 1, 4>;
using Flat2 = Shape<64, 128, 2, 2>;

template <class S, bool F16>
__device__ __forceinline__ void narrow_tile(const GroupLayer& ly, int sample, int tile, unsigned lds0, float* red,
                                            float* partial) {
  const int T = ly.T, d = ly.d_in, p = ly.d_out, nkb = (T + BK - 1) / BK;
  const int tiles_n = (p + S::BN - 1) / S::BN;
  const int m0 = (tile / tiles_n) * S::BM, n0 = (tile % tiles_n) * S::BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / S::WN) * 32, wn = (wave % S::WN) * (S::BN / S::WN);

  RowOperand<S::BM, 16> oa;
  RowOperand<S::BN, 16> ob;
  oa.init(static_cast<const uint16_t*>(ly.a) + (size_t)sample * T * d, T, d, m0, lds0, wave, lane);
  ob.init(static_cast<const uint16_t*>(ly.g) + (size_t)sample * T * p, T, p, n0, lds0 + S::A_BYTES, wave, lane);
  int p_stage = 0;
  auto issue = [&]() {
    oa.issue(p_stage * S::STAGE_BYTES, lane);
    ob.issue(p_stage * S::STAGE_BYTES, lane);
    p_stage = p_stage + 1 == NSTAGE ? 0 : p_stage + 1;
  };
  const unsigned a_rd = lds0 + row_frag_base<S::BM, 16>(wm, lane);
  unsigned b_rd[S::TN];
#pragma unroll
  for (int y = 0; y < S::TN; ++y) b_rd[y] = lds0 + S::A_BYTES + row_frag_base<S::BN, 16>(wn + 32 * y, lane);
  f32x16 acc[S::TN];
#pragma unroll
  for (int y = 0; y < S::TN; ++y)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[y][r] = 0.f;

  for (int q = 0; q < NSTAGE - 1; ++q) issue();
  int stage = 0;
  for (int kb = 0; kb < nkb; ++kb) {
    // own loads of block kb landed, own LDS reads of block kb - 1 done; then everyone's
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NSTAGE - 2) * S::LOADS) : "memory");
    issue();
    const unsigned so = stage * S::STAGE_BYTES;
    bf16x8 fa[2], fb[2][S::TN];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      fa[ks] = read_row_frag<S::BM>(a_rd + so + ks * 16 * S::BM * 2);
#pragma unroll
      for (int y = 0; y < S::TN; ++y) fb[ks][y] = read_row_frag<S::BN>(b_rd[y] + so + ks * 16 * S::BN * 2);
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int y = 0; y < S::TN; ++y) acc[y] = mfma16<F16>(fb[ks][y], fa[ks], acc[y]);
    stage = stage + 1 == NSTAGE ? 0 : stage + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // zero-fill loads past the end
  __syncthreads();                                       // LDS is reused below

  // transposed layout, as in perex_dma.hip
  if (ly.out) {
    float* dst = ly.out + (size_t)sample * d * p;
    const int row = m0 + wm + (lane & 31);
#pragma unroll
    for (int y = 0; y < S::TN; ++y) {
      const int col0 = n0 + wn + 32 * y + 4 * (lane >> 5);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (row < d && col0 + 8 * q < p) {
          const f32x4v w = {acc[y][4 * q], acc[y][4 * q + 1], acc[y][4 * q + 2], acc[y][4 * q + 3]};
          *reinterpret_cast<f32x4v*>(dst + (size_t)row * p + col0 + 8 * q) = w;
        }
    }
  }
  float sum = 0.f;                                       // without the padding: an infinity beside it makes it NaN
  const bool in_rows = m0 + wm + (lane & 31) < d;
#pragma unroll
  for (int y = 0; y < S::TN; ++y)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float v = in_rows && n0 + wn + 32 * y + 8 * (r >> 2) + 4 * (lane >> 5) < p ? acc[y][r] : 0.f;
      sum = fmaf(v, v, sum);
    }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) red[wave] = sum;
  __syncthreads();
  if (tid == 0) *partial = (red[0] + red[1]) + (red[2] + red[3]);
}

template <bool F16>
__global__ void __launch_bounds__(NT)
perex_narrow_kernel(const GroupArgs ga, float* __restrict__ partials) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  // the tiles of one sample share its panels of the narrow operand
  const int item = contiguous_eighth(blockIdx.x, ga.total_blocks);
  const int l = layer_of(ga, item);
  const GroupLayer& ly = ga.layer[l];
  const int local = item - ly.tile_begin;
  const int sample = local / ly.tiles_per_sample, tile = local - sample * ly.tiles_per_sample;
  auto run = [&](auto shape) {
    narrow_tile<decltype(shape), F16>(ly, sample, tile, (unsigned)(uintptr_t)lds_raw,
                                      reinterpret_cast<float*>(lds_raw), partials + ly.part_begin + local);
  };
  if (ly.d_out <= 32)
    run(Tall{});
  else if (ly.d_in <= 32)
    run(Flat{});
  else if (ly.d_out <= 64)
    run(Tall2{});
  else
    run(Flat2{});
}

// Long samples of many tiles: half a compute unit's LDS each, so that two workgroups share it and not four.  An XCD's
// 128 workgroups would stream from twice as many samples at a time, which costs 5 to 7 % once the loads set the time
// (96 samples of 4096 tokens, 2048 x 16: 293 us, so 277; of 256 tokens four are better, 19 us against 22).
constexpr int kLongTokens = 1024, kLongTiles = 16, kHalfLds = 79 * 1024;

template <bool F16>
dp_status launch_t(const GroupArgs& ga, float* partials, hipStream_t s) {
  int lds = NSTAGE * Tall::STAGE_BYTES, tiles = 0, T = INT32_MAX;
  for (int j = 0; j < ga.n_layers; ++j) {
    const GroupLayer& ly = ga.layer[j];
    if (ly.d_in > 32 && ly.d_out > 32) lds = NSTAGE * Tall2::STAGE_BYTES;
    tiles = ly.tiles_per_sample > tiles ? ly.tiles_per_sample : tiles;
    T = ly.T < T ? ly.T : T;
  }
  if (T >= kLongTokens && tiles >= kLongTiles) {
    static ReadyTable ready;
    lds = kHalfLds;
    dp_status st = allow_big_lds(perex_narrow_kernel<F16>, lds, ready);
    if (st != DP_OK) return st;
  }
  hipLaunchKernelGGL(perex_narrow_kernel<F16>, dim3(ga.total_blocks), dim3(NT), lds, s, ga, partials);
  return hip_status(hipGetLastError());
}

}  // namespace

// One tile covers the narrow side, so the tiles and partial-sum slots of a sample are those of 128 x 128
// tiles (perex_tiles_per_sample).  32-bit byte offsets inside a sample's slab, bit 31 as the "fetch zeros"
// marker; the prefetch runs up to NSTAGE blocks past the last row without wrapping.
bool perex_narrow_supports(int T, int d, int p) {
  const int64_t rows = (int64_t)T + (NSTAGE + 1) * BK;
  return (d <= 64 || p <= 64) && rows * d * 2 < (int64_t)1 << 31 && rows * p * 2 < (int64_t)1 << 31;
}

dp_status launch_perex_narrow_group(const GroupArgs& ga, float* partials, hipStream_t s) {
  return ga.f16 ? launch_t<true>(ga, partials, s) : launch_t<false>(ga, partials, s);
}

}  // namespace dpbk
