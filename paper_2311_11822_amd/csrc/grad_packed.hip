// Clip-weighted gradient over packed token rows (section 3 of the paper, "DP gradient"), for short
// samples and for narrow layers:   grad[j,k] = sum_r C_{r / T} a[r,j] g[r,k],   r = 0 .. B T - 1.
//
// The kernels that keep the weights out of the operands (grad_gemm.hip, tn_tile.h) re-express
// their accumulator at every sample boundary and pad every sample to whole 32-row k-blocks: at T = 1
// that is all they do.  Here the rows of all samples form one contraction of B T rows and the weight
// is multiplied into the a operand in fp32; that product is then cut into three bfloat16 parts, whose
// sum is within 2^-25 of it, so each 32-row step takes three matrix instructions and less is lost than
// by rounding C a to fp32.  fp16 operands: g (11 bits) is cut into two bfloat16 parts exactly, six
// instructions.  They are 16x16x32 ones: the card's power holds the clock (1.25 GHz under 32x32x16), and they take less of it (gradients
// of eight layers 1024 x 1024, us, 32x32x16 and these: 512 x 1 token 27.3, 26.3; 256 x 16 177.4, 170.4; fp16 64 x 8 49.8, 47.9; 24 of
// 768 x 16, 512 x 32 260.0, 258.4).  Gradients measured against 64 bits: 1.4e-7 (T = 1, B = 512) and 2.1e-7 (T = 31) here,
// 6.0e-7 and 3.9e-7 in the large-tile kernel.
//   Measured, eight layers of 1024 x 1024 .. 4096 outputs, bf16: B = 512, T = 1: 1384 us before, 84 us here; 4096
// rows, T = 1 and 16: 565 us on 32x32x16 instructions, 530 here (what bounds it: the matrix cores at the clock that the power leaves,
// then the cutting); the large-tile kernel 684 us at T = 16, 352 at 32.
// packed_below (dp_api.hip) draws its lines there.
//
// Tiles (four waves, 32 gradient rows each where the layer is wide): 128 x 128, or 128 x 32, 128 x 64 and
// their transposes for layers narrower than a tile, where the stream over the wide operand is the bound and padding
// the narrow one to 128 would multiply its LDS traffic.  Operand rows go global -> LDS without passing
// through registers, four stages of 32 rows, three blocks in flight; the 32 rows' weights travel
// with them (a 4-byte gather of C by row / T).  Two workgroups share a compute unit: one's splitting
// runs beside the other's matrix instructions.
//
// Rows of a sample with C == 0 do not enter (whatever they hold): a wave that meets a zero weight clears
// those rows in both operands.
//
// Range.  The contract is that of weights applied to a sample's exact partial product, so no part of C a may be lost
// below the normal numbers: the weights are multiplied by 2^80 on their way in and the sums by 2^-80 at the
// end.  C a >= 2^-178 then keeps its parts (2^-98 scaled, 2^-126 the last part's end), which every weight of 2^-45
// and more does with every bfloat16 (2^-133 at least), and every weight with every fp16 (2^-24).  Where a smaller
// weight came by, or a sum is not finite (an infinity in an operand meets the zero low parts of the other; C a or
// sums beyond 2^48), the workgroup forms its tile again without the cutting: the same loads, the rows of one
// sample at a time, unweighted, folded in as total += C_i * sum.  (One wave on its own, two rows of its 32 x 32
// pieces at a time straight from memory, took 52.6 ms for 131072 rows of eight 768 x 16 layers; so 4.4, and 2.1
// where all is finite.)  The scaling, where each weight is used, and the test cost nothing measurable (4 % of a launch
// of a few workgroups).
#include <float.h>

#include "dp_internal.h"
#include "grad_epilogue.h"
#include "row_tile.h"
#include "tile_order.h"

namespace dpbk {

namespace {

constexpr int BK = 32, NSTAGE = 4, NT = 256;

// WM x WN waves over a BM x BN tile; each holds 32 rows x (BN / WN) columns.
template <int BM_, int BN_, int WM_, int WN_>
struct Shape {
  static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_;
  static constexpr int XM = 2, XN = BN / WN / 16;               // 16 x 16 tiles of a wave
  static constexpr int A_BYTES = BK * BM * 2, B_BYTES = BK * BN * 2;
  static constexpr int W_BYTES = 256;                          // weights of the 32 rows (twice)
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES + W_BYTES;
  static constexpr int LOADS = kRowLoads<BM> + kRowLoads<BN> + 1;                 // per wave per k-block
  static_assert(BM / WM == 32 && WM * WN == 4, "shape");
};
using Wide = Shape<128, 128, 4, 1>;
using Tall = Shape<128, 32, 4, 1>;
using Tall2 = Shape<128, 64, 4, 1>;
using Flat = Shape<32, 128, 1, 4>;
using Flat2 = Shape<64, 128, 2, 2>;
constexpr int FLAGS = NSTAGE * Wide::STAGE_BYTES;              // a word per wave behind the stages
constexpr int LDS_BYTES = FLAGS + 16;                          // 65 KiB: two workgroups per compute unit

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
constexpr float kScale = 0x1p80f;                             // of the weights: see "Range"
template <bool F16>
constexpr float kLeastWeight = F16 ? 0.f : 0x1p-45f;

template <bool F16>
__device__ __forceinline__ float widen_lo(uint32_t u) {
  return F16 ? (float)__builtin_bit_cast(_Float16, (uint16_t)(u & 0xFFFFu)) : __uint_as_float(u << 16);
}
template <bool F16>
__device__ __forceinline__ float widen_hi(uint32_t u) {
  return F16 ? (float)__builtin_bit_cast(_Float16, (uint16_t)(u >> 16)) : __uint_as_float(u & 0xFFFF0000u);
}
// The upper halves of two fp32 values as one pair of bfloat16 (truncation).
__device__ __forceinline__ uint32_t pack_hi(float x0, float x1) {
  return __builtin_amdgcn_perm(__float_as_uint(x1), __float_as_uint(x0), 0x07060302u);
}
__device__ __forceinline__ float top8(float x) { return __uint_as_float(__float_as_uint(x) & 0xFFFF0000u); }

// The products w x of a pair -> three pairs of bfloat16 parts, the highest first.  The remainder behind the
// first part is formed from the exact product and fits 24 bits; the last part is rounded to nearest.
__device__ __forceinline__ void cut_product(float w0, float x0, float w1, float x1, uint32_t (&part)[3]) {
  typedef __attribute__((ext_vector_type(2))) float f2;
  typedef __attribute__((ext_vector_type(2))) __bf16 b2;
  const float y0 = w0 * x0, y1 = w1 * x1;
  const float r0 = fmaf(w0, x0, -top8(y0)), r1 = fmaf(w1, x1, -top8(y1));
  const f2 last = {r0 - top8(r0), r1 - top8(r1)};
  part[0] = pack_hi(y0, y1);
  part[1] = pack_hi(r0, r1);
  part[2] = __builtin_bit_cast(uint32_t, __builtin_convertvector(last, b2));
}
// A pair of fp16 values (11 bits) -> two pairs of bfloat16 parts, exactly.
__device__ __forceinline__ void cut_f16(uint32_t u, uint32_t (&part)[2]) {
  const float x0 = widen_lo<true>(u), x1 = widen_hi<true>(u);
  part[0] = pack_hi(x0, x1);
  part[1] = pack_hi(x0 - top8(x0), x1 - top8(x1));
}

template <class S, bool F16, bool NOISE>
__device__ __forceinline__ void packed_tile(const GroupLayer& ly, int layer, int tile, int B, bool accumulate,
                                            const float* C, const NoiseArgs& na, unsigned lds0) {
  const int T = ly.T, d = ly.d_in, p = ly.d_out;
  int stream = ly.stream;
  asm volatile("" : "+s"(stream));                       // read with the rest of the layer, not in front of the first store
  const int tiles_n = (p + S::BN - 1) / S::BN;
  const int m0 = (tile / tiles_n) * S::BM, n0 = (tile % tiles_n) * S::BN;
  const int rows = B * T, nkb = (rows + BK - 1) / BK;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / S::WN) * 32, wn = (wave % S::WN) * (S::BN / S::WN);

  RowOperand<S::BM, 32> oa;
  RowOperand<S::BN, 32> ob;
  // weights: lane -> row (lane & 31) of the k-block, sample w_i and token w_t of that row
  const i32x4 rw = make_rsrc(C, (unsigned)B * 4u);
  int w_i, w_t;
  const int w_di = BK / T, w_dt = BK % T;
  int p_stage;
  auto rewind = [&]() {                                  // the load stream to the first k-block
    int x = lane;
    asm volatile("" : "+v"(x));                          // computed anew each time, not kept in registers through the loop
    oa.init(ly.a, rows, d, m0, lds0, wave, x);
    ob.init(ly.g, rows, p, n0, lds0 + S::A_BYTES, wave, x);
    w_i = (x & 31) / T;
    w_t = (x & 31) % T;
    p_stage = 0;
  };
  auto issue = [&]() {
    const unsigned so = p_stage * S::STAGE_BYTES;
    oa.issue(so, lane);
    ob.issue(so, lane);
    load_dword_to_lds(rw, (unsigned)w_i * 4u, lds0 + so + S::A_BYTES + S::B_BYTES);    // rows past the end: 0
    w_i += w_di;
    w_t += w_dt;
    if (w_t >= T) {
      w_t -= T;
      ++w_i;
    }
    p_stage = p_stage + 1 == NSTAGE ? 0 : p_stage + 1;
  };

  unsigned a_rd[S::XM], b_rd[S::XN];
#pragma unroll
  for (int x = 0; x < S::XM; ++x) a_rd[x] = lds0 + row_frag_base<S::BM, 32>(wm + 16 * x, lane);
#pragma unroll
  for (int y = 0; y < S::XN; ++y) b_rd[y] = lds0 + S::A_BYTES + row_frag_base<S::BN, 32>(wn + 16 * y, lane);
  const unsigned w_rd = lds0 + S::A_BYTES + S::B_BYTES + 32u * (lane >> 4);

  typedef __attribute__((ext_vector_type(4))) float f4;
  typedef __attribute__((address_space(3))) f4 lds_f4;
  typedef __attribute__((address_space(3))) float lds_float;
  constexpr int G_PARTS = F16 ? 2 : 1;
  // The products of the low parts go to sums of their own, whose roundings are 2^-8 of the others': the
  // result is rounded as often as one matrix instruction per step would.
  f32x4 acc[S::XM][S::XN], low[S::XM][S::XN];
  auto clear = [&]() {
#pragma unroll
    for (int x = 0; x < S::XM; ++x)
#pragma unroll
      for (int y = 0; y < S::XN; ++y) acc[x][y] = low[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();

  float least_w = INFINITY;                              // smallest non-zero weight that this lane met

  // No load is on its way here, but the compiler does not know: of the old values that another tile shape's epilogue asks for, which
  // in its flow graph comes before this one, it would wait for in every round of the loop, and so for all of the loop's own
  // (26 layers 24 x 48, 4621 x 22 tokens, without noise: 2774 us with that wait, 1604 without).
  __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0)
  rewind();
  for (int q = 0; q < NSTAGE - 1; ++q) issue();
  int stage = 0;
  for (int kb = 0; kb < nkb; ++kb) {
    // own loads of block kb landed, own LDS reads of block kb - 1 done; then everyone's
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NSTAGE - 2) * S::LOADS) : "memory");
    issue();
    const unsigned so = stage * S::STAGE_BYTES;
    const float own = *(const lds_float*)(uintptr_t)(lds0 + so + S::A_BYTES + S::B_BYTES + 4 * lane);  // row lane & 31
    u32x4 fa[S::XM], fb[S::XN];
    const lds_f4* wp = (const lds_f4*)(uintptr_t)(w_rd + so);
    f4 w[2] = {wp[0], wp[1]};                            // weights of this lane's 8 rows
#pragma unroll
    for (int x = 0; x < S::XM; ++x) fa[x] = __builtin_bit_cast(u32x4, read_row_frag<S::BM>(a_rd[x] + so));
#pragma unroll
    for (int y = 0; y < S::XN; ++y) fb[y] = __builtin_bit_cast(u32x4, read_row_frag<S::BN>(b_rd[y] + so));
    DP_PIN();
    least_w = own == 0.f ? least_w : fminf(least_w, fabsf(own));
    if (__any(own == 0.f)) {                             // rows that do not count (or lie past the end)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = 2 * q & 3;
        const f4 ww = w[q >> 1];
        const uint32_t m = (ww[e] == 0.f ? 0u : 0xFFFFu) | (ww[e + 1] == 0.f ? 0u : 0xFFFF0000u);
#pragma unroll
        for (int x = 0; x < S::XM; ++x) fa[x][q] &= m;
#pragma unroll
        for (int y = 0; y < S::XN; ++y) fb[y][q] &= m;
      }
    }
    w[0] *= kScale;
    w[1] *= kScale;
    // The second half's cutting fills the gaps between the first half's matrix instructions.
    u32x4 xa[S::XM][3], xb[S::XN][G_PARTS];
    auto cut = [&](int x) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f4 ww = w[q >> 1];
        const int e = 2 * q & 3;
        uint32_t part[3];
        cut_product(ww[e], widen_lo<F16>(fa[x][q]), ww[e + 1], widen_hi<F16>(fa[x][q]), part);
#pragma unroll
        for (int n = 0; n < 3; ++n) xa[x][n][q] = part[n];
      }
    };
    auto multiply = [&](int x) {
#pragma unroll
      for (int n = 2; n >= 0; --n)
#pragma unroll
        for (int m = G_PARTS - 1; m >= 0; --m)
#pragma unroll
          for (int y = 0; y < S::XN; ++y) {
            f32x4& sum = n + m ? low[x][y] : acc[x][y];
            sum = mfma16<false>(__builtin_bit_cast(bf16x8, xb[y][m]), __builtin_bit_cast(bf16x8, xa[x][n]), sum);
          }
    };
    cut(0);
#pragma unroll
    for (int y = 0; y < S::XN; ++y)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (F16) {
          uint32_t gp[2];
          cut_f16(fb[y][q], gp);
#pragma unroll
          for (int m = 0; m < G_PARTS; ++m) xb[y][m][q] = gp[m];
        } else {
          xb[y][0][q] = fb[y][q];
        }
      }
    DP_PIN();
    multiply(0);
    cut(1);
#pragma unroll
    for (int n = 0; n < 3 * G_PARTS * S::XN; ++n) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                       // one MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, F16 ? 3 : S::XN == 4 ? 5 : 2, 0);   // some vector-ALU instructions, as measured
    }
    DP_PIN();
    multiply(1);
    stage = stage + 1 == NSTAGE ? 0 : stage + 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // zero-fill loads past the end

  float largest = 0.f;                                   // NaN if a sum is
#pragma unroll
  for (int x = 0; x < S::XM; ++x)
#pragma unroll
    for (int y = 0; y < S::XN; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        acc[x][y][r] = (acc[x][y][r] + low[x][y][r]) * (1.f / kScale);
        largest = __builtin_elementwise_maximum(largest, fabsf(acc[x][y][r]));
      }
  const bool off = least_w < kLeastWeight<F16> || !(largest <= FLT_MAX);
  typedef __attribute__((address_space(3))) int lds_int;
  const bool wave_off = __any(off);
  if (lane == 0) *(lds_int*)(uintptr_t)(lds0 + FLAGS + 4 * wave) = wave_off;
  __syncthreads();                                       // nobody reads a stage any more either
  int any_off = 0;
#pragma unroll
  for (int v = 0; v < 4; ++v) any_off |= *(lds_int*)(uintptr_t)(lds0 + FLAGS + 4 * v);
  if (__builtin_amdgcn_readfirstlane(any_off)) {
    // The tile again, unweighted, sample by sample (low: the sample's sum so far).
    clear();
    rewind();
    for (int q = 0; q < NSTAGE - 1; ++q) issue();
    stage = 0;
    int left = T;                                        // rows of the sample from here on
    for (int kb = 0; kb < nkb; ++kb) {
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"((NSTAGE - 2) * S::LOADS) : "memory");
      issue();
      const unsigned so = stage * S::STAGE_BYTES;
      u32x4 fa[S::XM], fb[S::XN];
#pragma unroll
      for (int x = 0; x < S::XM; ++x) fa[x] = __builtin_bit_cast(u32x4, read_row_frag<S::BM>(a_rd[x] + so));
#pragma unroll
      for (int y = 0; y < S::XN; ++y) fb[y] = __builtin_bit_cast(u32x4, read_row_frag<S::BN>(b_rd[y] + so));
      const int here = min(BK, rows - kb * BK);
#pragma unroll 1
      for (int begin = 0; begin < here;) {
        const int end = min(here, begin + left);
        const int c_bits = *(const lds_int*)(uintptr_t)(lds0 + so + S::A_BYTES + S::B_BYTES + 4 * begin);
        const float c = __int_as_float(__builtin_amdgcn_readfirstlane(c_bits));
        if (c != 0.f) {
          u32x4 keep;                                    // this lane's rows 8 (lane >> 4) + 0 .. 7
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int row = 8 * (lane >> 4) + 2 * q;
            keep[q] = (row >= begin && row < end ? 0xFFFFu : 0u) |
                      (row + 1 >= begin && row + 1 < end ? 0xFFFF0000u : 0u);
          }
#pragma unroll
          for (int x = 0; x < S::XM; ++x)
#pragma unroll
            for (int y = 0; y < S::XN; ++y)
              low[x][y] = mfma16<F16>(__builtin_bit_cast(bf16x8, fb[y] & keep), __builtin_bit_cast(bf16x8, fa[x] & keep), low[x][y]);
        }
        left -= end - begin;
        begin = end;
        if (left == 0) {
          left = T;
          if (c != 0.f) {
#pragma unroll
            for (int x = 0; x < S::XM; ++x)
#pragma unroll
              for (int y = 0; y < S::XN; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  acc[x][y][r] = fmaf(c, low[x][y][r], acc[x][y][r]);
                  low[x][y][r] = 0.f;
                }
          }
        }
      }
      stage = stage + 1 == NSTAGE ? 0 : stage + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // zero-fill loads past the end
    __syncthreads();
  }

  // epilogue; nobody reads a stage any more
  TileNoise tn = {};
  if (NOISE) tn = load_tile_noise(na, layer);
  constexpr int NY = S::XN == 2 ? 1 : 2;
  using Piece = WavePiece16<NY, 32, S::XN>;
  static_assert(Piece::BYTES * 4 <= NSTAGE * S::STAGE_BYTES && S::XM == 2, "a region for each wave");
  store_pieces<S::XN / (2 * NY), F16, NOISE, false>(
      [&](int y) { return Piece{&acc[0][2 * NY * y], m0 + wm, n0 + wn + 32 * NY * y}; }, accumulate, stream, 1.f,
      lds0 + wave * Piece::BYTES, ly.out, d, p, tn, lane, []() {});
}

// GroupLayer::path holds the layer's tile shape (packed_shape).
template <bool F16, bool NOISE>
__global__ void __launch_bounds__(NT, 2)
grad_packed_kernel(const GroupArgs ga, const float* __restrict__ C_all, const NoiseArgs na) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  const unsigned lds0 = (unsigned)(uintptr_t)lds_raw;
  // Tiles of one row share a panel of a: runs of 32 consecutive numbers meet in one XCD's L2.  (Not
  // an eighth of the launch each: a shard's noise lies in consecutive tiles and would land on few XCDs;
  // a step of eight layers, B = 512, T = 1, noise on an eighth of 12.6 M elements: 131 us against 140.)
  const int item = grad_logical_tile(blockIdx.x, ga.total_blocks);
  const int l = layer_of(ga, item);
  const GroupLayer& ly = ga.layer[l];
  const float* C = C_all + ly.c_off;
  const int tile = item - ly.tile_begin;
  auto run = [&](auto shape) {
    packed_tile<decltype(shape), F16, NOISE>(ly, l, tile, ga.B, ga.accumulate, C, na, lds0);
  };
  switch (ly.path) {
    case 0: run(Wide{}); break;
    case 1: run(Tall{}); break;
    case 2: run(Flat{}); break;
    case 3: run(Tall2{}); break;
    default: run(Flat2{});
  }
}

template <bool F16, bool NOISE>
dp_status launch_t(const GroupArgs& ga, const float* C, const NoiseArgs& na, hipStream_t s) {
  auto kernel = grad_packed_kernel<F16, NOISE>;
  static ReadyTable ready;
  dp_status st = allow_big_lds(kernel, LDS_BYTES, ready);
  if (st != DP_OK) return st;
  hipLaunchKernelGGL(kernel, dim3(ga.total_blocks), dim3(NT), LDS_BYTES, s, ga, C, na);
  return hip_status(hipGetLastError());
}

int tiles_of(int d, int p, int bm, int bn) { return ((d + bm - 1) / bm) * ((p + bn - 1) / bn); }

}  // namespace

// A layer of up to 64 columns (rows) takes a tile that covers that side, so the other operand is read once.
int grad_packed_shape(int d, int p) { return p <= 32 ? 1 : d <= 32 ? 2 : p <= 64 ? 3 : d <= 64 ? 4 : 0; }

int grad_packed_tiles(int d, int p) {
  switch (grad_packed_shape(d, p)) {
    case 1: return tiles_of(d, p, Tall::BM, Tall::BN);
    case 2: return tiles_of(d, p, Flat::BM, Flat::BN);
    case 3: return tiles_of(d, p, Tall2::BM, Tall2::BN);
    case 4: return tiles_of(d, p, Flat2::BM, Flat2::BN);
    default: return tiles_of(d, p, Wide::BM, Wide::BN);
  }
}

// All rows of an operand through one descriptor with 32-bit byte offsets; the prefetch runs up to
// NSTAGE blocks past the last row without wrapping.
bool grad_packed_supports(int B, int T, int d, int p) {
  const int64_t rows = (int64_t)B * T + (NSTAGE + 1) * BK;
  return rows * d * 2 < (int64_t)1 << 31 && rows * p * 2 < (int64_t)1 << 31;
}

dp_status launch_grad_packed_group(const GroupArgs& ga, const float* C, const NoiseArgs* noise, hipStream_t s) {
  static const NoiseArgs none = {};
  const NoiseArgs& na = noise ? *noise : none;
  switch ((ga.f16 ? 2 : 0) + (noise ? 1 : 0)) {
    case 0: return launch_t<false, false>(ga, C, na, s);
    case 1: return launch_t<false, true>(ga, C, na, s);
    case 2: return launch_t<true, false>(ga, C, na, s);
    default: return launch_t<true, true>(ga, C, na, s);
  }
}

}  // namespace dpbk
