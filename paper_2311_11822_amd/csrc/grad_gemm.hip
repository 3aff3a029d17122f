// Clip-weighted gradient on the matrix cores (section 3 of the paper,
// "DP gradient"):   grad[j,k] = sum_i C_i sum_t a[i,t,j] g[i,t,k].
//
// 256 x 256 output tiles, one workgroup per compute unit (contraction: tn_weighted.h, tn_pipeline.h), and 128 x 128
// or 64 x 64 ones for the end of a launch and for launches that would leave compute units idle.
#include <type_traits>

#include "dp_internal.h"
#include "grad_epilogue.h"
#include "tile_order.h"
#include "tn_pipeline.h"
#include "tn_weighted.h"

namespace dpbk {

namespace {

constexpr int BM = BigTile::BM, BN = BigTile::BN;

// Tile t of the launch, one of layer l's -> tile origin (order inside a layer: tile_order.h).
__device__ __forceinline__ void locate_tile(const GroupArgs& ga, int l, int t, int& m0, int& n0) {
  const GroupLayer& ly = ga.layer[l];
  int tm, tn;
  grad_tile_of((ly.d_in + BM - 1) / BM, (ly.d_out + BN - 1) / BN, t - ly.tile_begin, tm, tn);
  m0 = tm * BM;
  n0 = tn * BN;
}

template <class S, bool F16, bool NOISE, bool OUT16>
__device__ __forceinline__ void gradient_tile(const GroupArgs& ga, int l, int m0, int n0, const float* C, float w,
                                              const NoiseArgs& na) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  const GroupLayer& ly = ga.layer[l];
  const int d = ly.d_in, p = ly.d_out;
  f32x16 acc[S::TM][S::TN];
  const float held = tn_contract<S, F16, true>(ly.a, ly.g, ly.T, d, p, 0, ga.B, C, w, m0, n0,
                                               (unsigned)(uintptr_t)lds_raw, acc);

  // epilogue: grad (+)= held * acc (+ noise).  With no active sample the accumulator is zero.
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int wm = (wave / S::WN) * S::WTM, wn = (wave % S::WN) * S::WTN;
  using Piece = WavePiece<S::TN>;
  static_assert(Piece::BYTES * S::WM * S::WN <= S::LDS_BYTES, "a region for each wave");
  const unsigned region = (unsigned)(uintptr_t)lds_raw + wave * Piece::BYTES;
  TileNoise tn = {};
  if (NOISE) tn = load_tile_noise(na, l);
  __syncthreads();                                     // the last fragments are read
  store_pieces<S::TM, F16, NOISE, OUT16>([&](int x) { return Piece{acc[x], m0 + wm + x * 32, n0 + wn}; }, ga.accumulate, ly.stream, held,
                                         region, ly.out, d, p, tn, lane, []() {});
}

template <bool F16, bool NOISE, bool OUT16>
__global__ void __launch_bounds__(BigTile::NT)
clipped_grad_big_kernel(const GroupArgs ga, const float* __restrict__ C_all, const NoiseArgs na) {
  const int logical = grad_logical_tile(blockIdx.x, ga.total_blocks);     // XCD-aware: tile_order.h
  const int l = layer_of(ga, logical);
  const float* C = C_all + ga.layer[l].c_off;                             // the layer's clipping group
  const float w = window_weights(C, 0, ga.B);
  int m0, n0;
  locate_tile(ga, l, logical, m0, n0);
  gradient_tile<BigTile, F16, NOISE, OUT16>(ga, l, m0, n0, C, w, na);
}

// Epilogue of the kernels of whole k-blocks.
template <class S, bool F16, bool NOISE, bool OUT16>
struct StoreTile {
  const GroupArgs& ga;
  const NoiseArgs& na;
  template <class Ready>
  __device__ __forceinline__ void operator()(const WeightedTile& t, const f32x4 (&acc)[S::WTM / 16][S::WTN / 16], float held,
                                             unsigned region, int wm, int wn, Ready ready) const {
    using Piece = WavePiece16<2, 16, 4>;
    static_assert(Piece::BYTES * S::WM * S::WN <= S::STAGE_BYTES, "a region for each wave");
    const GroupLayer& ly = ga.layer[t.l];
    TileNoise tn = {};
    if (NOISE) tn = load_tile_noise(na, t.l);
    store_pieces<S::WTM / 16, F16, NOISE, OUT16>(
        [&](int x) { return Piece{&acc[x][0], t.m0 + wm + x * 16, t.n0 + wn}; }, ga.accumulate, ly.stream, held, region, ly.out,
        ly.d_in, ly.d_out, tn, threadIdx.x & 63, ready);
  }
};

struct BigTiles {
  int total;
  __device__ __forceinline__ int tile(int id) const { return grad_logical_tile(id, total); }
  __device__ __forceinline__ bool operator()(const GroupArgs& ga, WeightedTile& t, int id) const {
    locate_tile(ga, t.l, tile(id), t.m0, t.n0);
    return true;
  }
};

template <bool F16, bool NOISE, bool OUT16>
__global__ void __launch_bounds__(BigTile::NT)
clipped_grad_blocks_kernel(const GroupArgs ga, const float* __restrict__ C_all, const NoiseArgs na) {
  weighted_tiles<BigTile, F16, true>(ga, C_all, blockIdx.x, gridDim.x, ga.total_blocks, BigTiles{ga.total_blocks},
                                     StoreTile<BigTile, F16, NOISE, OUT16>{ga, na});
}

// End of a launch.  All tiles of a launch take the same time and one workgroup fills a compute
// unit, so n tiles run in ceil(n / 256) rounds; what the last round would hold is cut into 128 x 128
// sub-tiles where these fill the chip better (clipped_grad_tail), in the order of grad_sub_tile.  The k-steps of an output element are added in the same order as
// in the kernel above: the same bits.
constexpr int MID_SIDE = kGradMidSide, MID_SUBS = MID_SIDE * MID_SIDE;
static_assert(MID_SIDE * MidTile::BM == BM && MID_SIDE * MidTile::BN == BN, "sub-tiles of a tile");

template <class S, bool F16, bool NOISE, bool OUT16>
__global__ void __launch_bounds__(S::NT, 163840 / S::LDS_BYTES)
clipped_grad_mid_kernel(const GroupArgs ga, const float* C_all, int first_tile, const NoiseArgs na) {
  const SubTile sub = grad_sub_tile<MID_SIDE>(blockIdx.x, gridDim.x);
  const int l = layer_of(ga, first_tile + sub.tile);
  const float* C = C_all + ga.layer[l].c_off;
  const float w = first_weights(C, ga.B);
  int m0, n0;
  locate_tile(ga, l, first_tile + sub.tile, m0, n0);
  m0 += sub.row * MidTile::BM;
  n0 += sub.col * MidTile::BN;
  if (m0 >= ga.layer[l].d_in || n0 >= ga.layer[l].d_out) return;      // past the layer's edge (whole workgroup)
  gradient_tile<S, F16, NOISE, OUT16>(ga, l, m0, n0, C, w, na);
}

struct MidTiles {
  int first_tile;
  __device__ __forceinline__ SubTile sub(int id) const { return grad_sub_tile<MID_SIDE>(id, gridDim.x); }
  __device__ __forceinline__ int tile(int id) const { return first_tile + sub(id).tile; }
  __device__ __forceinline__ bool operator()(const GroupArgs& ga, WeightedTile& t, int id) const {
    locate_tile(ga, t.l, tile(id), t.m0, t.n0);
    t.m0 += sub(id).row * MidTile::BM;
    t.n0 += sub(id).col * MidTile::BN;
    return t.m0 < ga.layer[t.l].d_in && t.n0 < ga.layer[t.l].d_out;
  }
};

template <class S, bool F16, bool NOISE, bool OUT16>
__global__ void __launch_bounds__(S::NT, 163840 / S::LDS_BYTES)
clipped_grad_mid_blocks_kernel(const GroupArgs ga, const float* C_all, int first_tile, const NoiseArgs na) {
  weighted_tiles<S, F16, false>(ga, C_all, blockIdx.x, gridDim.x, gridDim.x, MidTiles{first_tile},
                                StoreTile<S, F16, NOISE, OUT16>{ga, na});
}

// The last few tiles of a launch are cut finer still, into 64 x 64 sub-tiles of one small workgroup each, which spreads them
// over the whole chip.
constexpr int TAIL = SmallTile::BM, TAIL_SIDE = kGradTailSide, SUBS = TAIL_SIDE * TAIL_SIDE;
static_assert(TAIL_SIDE * TAIL == BM && BM == BN, "sub-tile shape");

template <bool F16, bool NOISE, bool OUT16>
__global__ void __launch_bounds__(SmallTile::NT, 2)
clipped_grad_tail_kernel(const GroupArgs ga, const float* __restrict__ C_all, int first_tile,
                         const NoiseArgs na) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  const unsigned lds0 = (unsigned)(uintptr_t)lds_raw;
  const SubTile sub = grad_sub_tile<TAIL_SIDE>(blockIdx.x, gridDim.x);
  const int l = layer_of(ga, first_tile + sub.tile);
  const GroupLayer& ly = ga.layer[l];
  const float* C = C_all + ly.c_off;
  const float w = first_weights(C, ga.B);
  int m0, n0;
  locate_tile(ga, l, first_tile + sub.tile, m0, n0);
  m0 += sub.row * TAIL;
  n0 += sub.col * TAIL;
  if (m0 >= ly.d_in || n0 >= ly.d_out) return;       // sub-tile past the layer's edge (whole workgroup)
  f32x4 acc[2][2];
  const float held = tn_weighted_small<F16>(ly, ga.B, C, w, m0, n0, lds0, acc);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  TileNoise tn = {};
  if (NOISE) tn = load_tile_noise(na, l);
  __syncthreads();                                   // the last fragments are read
  using Piece = WavePiece16<1, 32, 2>;
  // streaming: at most 32 tiles of a launch, 1.00 of the time either way
  store_pieces<1, F16, NOISE, OUT16>([&](int) { return Piece{&acc[0][0], m0 + 32 * (wave >> 1), n0 + 32 * (wave & 1)}; },
                                     ga.accumulate, true, held, lds0 + wave * Piece::BYTES, ly.out, ly.d_in, ly.d_out, tn,
                                     threadIdx.x & 63, []() {});
}

}  // namespace

int clipped_grad_big_tiles(int d, int p) { return ((d + BM - 1) / BM) * ((p + BN - 1) / BN); }

// The kernels address each sample's slab of a layer with 32-bit byte offsets and use bit 31 as
// the "fetch zeros" marker; offsets run up to the end of the last, perhaps partial, k-block.
bool clipped_grad_big_supports(int T, int d, int p) {
  const int64_t rows = ((int64_t)T + BigTile::BK - 1) / BigTile::BK * BigTile::BK;
  return rows * d * 2 < (int64_t)1 << 31 && rows * p * 2 < (int64_t)1 << 31;
}

int64_t clipped_grad_mid_tiles(int d, int p) {
  return ((int64_t)d + MidTile::BM - 1) / MidTile::BM * (((int64_t)p + MidTile::BN - 1) / MidTile::BN);
}

// The tiles of the last round go to sub-tiles where they fit one round of 128 x 128.  K = 4096, alone: 64 tiles 91 us
// as they are, 46 as sub-tiles; 128 tiles 98 and 73; 160 tiles 102 and 112.  All tiles do where that takes fewer
// rounds' time, because of the layers' edges (which sub-tiles leave out).
// Up to kTailMax tiles are cut into 64 x 64: 16 tiles of K = 4096 take 27 us so, 41 us in 128 x 128; 32 tiles 37 and 42; 48
// tiles 55 and 43; 64 tiles 64 and 46.  More than kTailUnits have two workgroups on some unit, which load half as fast each; where
// rows begin off 64-byte pieces of memory, 128 x 128 tiles are faster then from 4096 rows on: 39 x 1408 tokens, 17 layers 168 x 168 663
// and 481, 4 x 1024, two 1000 x 1000 44.1 and 38.7, 5 x 3540, 24 of 232 x 232 234 and 213; not of rows on 64-byte pieces (4 x 1024, 19 of 224 x
// 224 35.8 and 37.8), of 2048 rows with noise (0.94 to 1.05 of the time) or of short samples (64 x 100, 17 of 168 x 168 63.6 and 80.2; 16 x 300 45.9, 48.4;
// 32 x 384 111.4, 110.7).
// Short contractions (rows: of all samples, each rounded up to 32, as these lines were measured) are bound by the
// epilogue, which a large tile has a compute unit to itself for: 128 x 128, two to a unit, unless large ones come in whole
// rounds.  One sample: two layers 3744 x 2352 33.2 us mixed, 24.7 on 128 x 128 (before: 29); 17 of 33 tokens 76 and 69;
// 16 of 100 104 and 104; four layers 4096 x 4096 (four whole rounds) 62 and 66; 24 of 768 x 3072 64 and 59, three of 40
// tokens 79 and 80.
//
// Short contractions of more 128 x 128 tiles than have a place at two to a compute unit take three to a unit, of three
// stages each, where these are estimated to be through first: a round of 256 large tiles takes 12 us and 1 for each begun 32
// rows, 768 small ones 8.5 and 1.15 (16-bit gradients: 8.2 and 1.05, 5.2 and 1).  What they gain is that the fixed part of
// a tile (its lookup, first loads, noise and stores) runs beside other tiles' contraction; what they lose is operands read
// twice as often.  Gradients, us, large and 128 x 128 of five stages, 128 x 128 of three: one sample of 32 tokens, 16 layers of
// width 1472 100, 79, with noise 140, 107, in 16 bits 69, 53; four of 32, 24 layers of width 768 44, 40, with noise 60, 53; eight
// 56, 51 and 73, 66; eight of 32, 16 layers of width 808 52, 46 and 66, 60; above the line 16 x 32, width 768 84, 83; eight,
// width 1472 144, 166.  (The kernels have changed since: of 874 launches of 40 to 528 large tiles and 32 to 512 rows, with
// noise, without and in 16 bits, what these lines take is within 5 % of the fastest of the three in all but the next rule's and 11.)
//
// A single round of large tiles is through before small ones that take a second round of 768.  From 257 rows on, large and three to a
// unit, us: 16 x 32 tokens, 24 layers 768 x 768 with noise 31.1, 38.4; 8 x 64, 16 of 808 x 808 31.6, 39.8; 8 x 64, one 3744 x 3744 without
// noise 26.6, 31.1; of 208 to 240 tiles 6 to 21 %.  Up to 256 rows, with noise on an eighth, 20 % slower to 3 % faster; 8 x 64,
// three 2048 x 2048 (192 tiles, 768 small ones) 29.8, 26.8.
GradTail clipped_grad_tail(int n, int64_t n_mid, int64_t rows, bool whole_lines, bool long_off_sectors, bool out16) {
  constexpr int kTailMax = 32, kTailUnits = 16, kTailRows = 4096, kShortRows = 512, kOneRoundRows = 256;
  constexpr int kBriefMost = 1 << 20;                    // of these launch workgroups of 256 threads
  constexpr int64_t kBriefRound = 768;
  int tail = n % kBigRound;
  const bool crowded = n_mid > kMidRound && rows <= kShortRows && n <= kBriefMost;
  if (n <= kBigRound && n_mid > kBriefRound && rows > kOneRoundRows) return {0, TAIL_SIDE, false};
  if (n > kTailMax && tail != 0 && rows * (n < kBigRound ? 1 : n / kBigRound) <= kShortRows) return {n, MID_SIDE, crowded};
  if (crowded) {
    const int64_t blocks = (rows + BigTile::BK - 1) / BigTile::BK;
    const int64_t big = out16 ? 820 + 105 * blocks : 1200 + 100 * blocks, brief = out16 ? 520 + 100 * blocks : 850 + 115 * blocks;
    const int64_t rounds10 = n / kBigRound * 10 + (tail == 0 ? 0 : tail * MID_SUBS <= kMidRound ? 6 : 10);
    if (brief * std::max(n_mid, kBriefRound) * 10 < big * rounds10 * kBriefRound) return {n, MID_SIDE, true};
  }
  if (tail * MID_SUBS > kMidRound) tail = 0;
  // A round of small tiles in tenths of a large round's time.  Rows that are not whole 128-byte lines of memory cost them half
  // as many lines again (large tiles a quarter), and the longer the contraction the less of that L2 has at hand: 16 layers
  // 1024 x 1024 0.56 at 2048 rows and 0.64 at 8192, 1016 x 1016 0.65 and 0.76; nine 784 x 2352 .. 3136 in fp16, 10638 rows, 520 us
  // on large tiles and 767 on small ones; 16 of 520 x 1560 .. 2080, 16384 rows, 655 and 1024; eight of 1000 x 3000 .. 4000,
  // 4096 rows, 211 and 265.
  const int64_t mid_cost = whole_lines || rows <= 2048 ? 6 : rows <= 8192 ? 8 : 10;
  const int64_t mixed = (int64_t)(n / kBigRound) * 10 + (tail ? mid_cost : n % kBigRound ? 10 : 0);
  if (mid_cost * ((n_mid + kMidRound - 1) / kMidRound) < mixed) tail = n;
  const int small = long_off_sectors && rows >= kTailRows ? kTailUnits : kTailMax;
  return {tail, tail <= small ? TAIL_SIDE : MID_SIDE, false};
}

// The kernels of tn_weighted.h, whose samples take whole k-blocks of 32 rows, where the rows that are zeros cost less than 16x16x32
// matrix instructions gain.  Gradients with noise, us, 16-row steps of 32x32x16 and whole k-blocks: samples that fill an even
// number of 16-row steps: 8 x 64 tokens, 20 layers of width 896 40.7, 39.9; 16 x 64 69.7, 64.0; 8 x 96, six of width 2048 64.6, 60.4;
// 16 x 256, twelve 512 x 512 43.1, 41.2; one sample of 64 tokens 21.3, 21.9; one k-block a sample: 64 x 32, 24 of width 1280
// 207, 217.  An odd number: 32 x 48, 24 of width 1280 170, 185; 20 x 80 160, 169; 24 x 144, 32 of width 1024 245, 254; 10 x 176, 24 of
// width 1280 161, 163; 32 x 197, 48 of width 768 1072, 1079; 3 x 240, 20 of width 896 47.8, 48.0; 8 x 240, 24 of width 1280 169.3, 167.5.
// (Odd numbers of 15 to 29 steps, six stacks of 4096 rows and their ratios: with noise 0.96 to 1.04, on average 1.01; without 0.96 to 1.02, 0.99.)
bool whole_blocks(int B, int T) {
  const int steps = (T + 15) / 16;
  return (int64_t)B * T > 128 && steps >= (steps % 2 == 0 ? 4 : 15);
}

GradLaunches clipped_grad_launches(const GroupArgs& ga, bool out16) {
  constexpr int kLongSample = 384;                       // tokens (clipped_grad_tail)
  const int n = ga.total_blocks;
  int64_t n_mid = 0, rows = 0;
  bool whole_lines = true, off_sectors = false, no_short = true, one_length = true, blocks = true;
  for (int j = 0; j < ga.n_layers; ++j) {
    const GroupLayer& ly = ga.layer[j];
    n_mid += clipped_grad_mid_tiles(ly.d_in, ly.d_out);
    whole_lines = whole_lines && ly.d_in % 64 == 0 && ly.d_out % 64 == 0;
    off_sectors = off_sectors || ly.d_in % 32 != 0 || ly.d_out % 32 != 0;
    no_short = no_short && ly.T >= kLongSample;
    one_length = one_length && ly.T == ga.layer[0].T;
    blocks = blocks && whole_blocks(ga.B, ly.T);
    const int64_t r = (int64_t)ga.B * ((ly.T + BigTile::BK - 1) / BigTile::BK) * BigTile::BK;
    rows = r > rows ? r : rows;
  }
  const GradTail cut = clipped_grad_tail(n, n_mid, rows, whole_lines, off_sectors && no_short, out16);
  const int n_big = n - cut.tiles;
  // Large tiles on part of the chip alone (from 129 on: fewer are cut) are not held by its power, and 16-row steps take fewer clocks;
  // nor is a single round of a short contraction.  Whole k-blocks to steps, ratios of times with noise and without: up to 1024 rows 144 and
  // 160 tiles 1.01 to 1.07 and 1.00 to 1.04, 176 to 252 tiles 0.99 to 1.08 and 0.97 to 1.02; 2048 rows 1.00 to 1.06 and 1.00 to 1.05, 0.96
  // to 1.05 and 0.96 to 1.00; 4096 rows 0.99 to 1.02 and 0.98 to 1.02, 0.94 to 1.02 and 0.94 to 0.99.  (128 x 128 tiles on part of the
  // chip, two to a unit and with their noise beside each other's contraction: 0.92 to 1.02 of samples of an even number of steps.)
  constexpr int kPartOfTheChip = 160, kShortRound = 1024;
  if (cut.tiles == 0 && n <= (rows <= kShortRound ? kBigRound : kPartOfTheChip)) blocks = false;
  // Workgroups that go from tile to tile take equal numbers of them: for tiles of one length.
  return {cut, blocks, blocks && one_length && ga.B <= 64 ? std::min(n_big, kBigRound) : n_big};
}

template <bool F16, bool NOISE, bool OUT16>
dp_status launch_clipped_grad_big_group_t(const GroupArgs& ga, const float* C, const NoiseArgs& na,
                                          hipStream_t s) {
  const GradLaunches plan = clipped_grad_launches(ga, OUT16);
  const GradTail cut = plan.cut;
  const bool blocks = plan.blocks;
  const int n = ga.total_blocks, n_tail = cut.tiles;
  auto big = blocks ? clipped_grad_blocks_kernel<F16, NOISE, OUT16> : clipped_grad_big_kernel<F16, NOISE, OUT16>;
  auto mid = blocks ? clipped_grad_mid_blocks_kernel<MidTile, F16, NOISE, OUT16> : clipped_grad_mid_kernel<MidTile, F16, NOISE, OUT16>;
  auto brief =
      blocks ? clipped_grad_mid_blocks_kernel<ShortTile, F16, NOISE, OUT16> : clipped_grad_mid_kernel<ShortTile, F16, NOISE, OUT16>;
  auto tail = clipped_grad_tail_kernel<F16, NOISE, OUT16>;
  static ReadyTable ready_big[2], ready_mid[2], ready_tail;
  dp_status st = allow_big_lds(big, BigTile::LDS_BYTES, ready_big[blocks]);
  if (st == DP_OK) st = allow_big_lds(mid, MidTile::LDS_BYTES, ready_mid[blocks]);
  if (st == DP_OK) st = allow_big_lds(tail, SmallTile::LDS_BYTES, ready_tail);
  if (st != DP_OK) return st;
  if (n > n_tail) {
    GroupArgs main_args = ga;
    main_args.total_blocks = n - n_tail;
    hipLaunchKernelGGL(big, dim3(plan.workgroups), dim3(BigTile::NT), BigTile::LDS_BYTES, s, main_args, C, na);
    st = hip_status(hipGetLastError());
    if (st != DP_OK) return st;
  }
  if (n_tail == 0) return DP_OK;
  if (cut.side == TAIL_SIDE)
    hipLaunchKernelGGL(tail, dim3(n_tail * SUBS), dim3(SmallTile::NT), SmallTile::LDS_BYTES, s, ga, C, n - n_tail, na);
  else if (cut.brief)
    hipLaunchKernelGGL(brief, dim3(n_tail * MID_SUBS), dim3(ShortTile::NT), ShortTile::LDS_BYTES, s, ga, C, n - n_tail, na);
  else
    hipLaunchKernelGGL(mid, dim3(n_tail * MID_SUBS), dim3(MidTile::NT), MidTile::LDS_BYTES, s, ga, C, n - n_tail, na);
  return hip_status(hipGetLastError());
}

// out16: the layers' `out` pointers address 16-bit arrays of the operands' storage type.
dp_status launch_clipped_grad_big_group(const GroupArgs& ga, const float* C, const NoiseArgs* noise,
                                        hipStream_t s, bool out16) {
  static const NoiseArgs none = {};
  const NoiseArgs& na = noise ? *noise : none;
  switch ((ga.f16 ? 4 : 0) + (noise ? 2 : 0) + (out16 ? 1 : 0)) {
    case 0: return launch_clipped_grad_big_group_t<false, false, false>(ga, C, na, s);
    case 1: return launch_clipped_grad_big_group_t<false, false, true>(ga, C, na, s);
    case 2: return launch_clipped_grad_big_group_t<false, true, false>(ga, C, na, s);
    case 3: return launch_clipped_grad_big_group_t<false, true, true>(ga, C, na, s);
    case 4: return launch_clipped_grad_big_group_t<true, false, false>(ga, C, na, s);
    case 5: return launch_clipped_grad_big_group_t<true, false, true>(ga, C, na, s);
    case 6: return launch_clipped_grad_big_group_t<true, true, false>(ga, C, na, s);
    default: return launch_clipped_grad_big_group_t<true, true, true>(ga, C, na, s);
  }
}

}  // namespace dpbk
