// Token contraction of one output tile, shared by the clip-weighted gradient (grad_gemm.hip) and the
// instantiated norm (perex_dma.hip):   acc[j,k] = sum_i w_i sum_t a[i,t,j] g[i,t,k].
//
// Design for gfx950 (measured on the device: dense bf16 MFMA sustains 2.2 PFLOP/s; the
// transposing 64-bit LDS read sustains ~130-150 B/clk/CU, half the rate of 128-bit reads):
//  * Square tiles: 256 x 256 by eight waves of 128 x 64 (six fragment reads per eight MFMAs; all of the CU's LDS),
//    or 128 x 128 by four waves of 64 x 64 (four per four; two workgroups per CU).  A wave holds its
//    accumulators in ordinary registers next to its fragments.  Four waves of 128 x 128, measured before,
//    read less LDS per MFMA, but their 256 accumulators sit in accumulator registers, which the vector ALU
//    reaches only through copies: re-expressing them at a sample boundary (below) cost ~4400 clocks
//    against ~1400 per 32 tokens, here ~600.  Eight 1024-wide layers (gradient stage): 64 x 64 tokens 410 ->
//    268 us, 32 x 128 316 -> 240; 12 GPT blocks of width 768, 16 x 256 tokens 780 -> 704, of 1280, 8 x 512
//    1863 -> 1787; at 2048 tokens 3 % faster.
//  * global -> LDS without passing through registers (buffer_load ... lds, 16 B per lane).
//    A wave's load lands as 1 KiB of consecutive LDS = two 512-byte (four 256-byte) k rows, so rows cannot be
//    padded; instead the 16-byte chunks of row k are XOR-swizzled by (k & 3) << 2, which
//    spreads four consecutive k rows over the four 64-byte bank groups the transposing read
//    touches at once.  Out-of-range chunks (tile edge, rows past the end of a sample whose T is no multiple
//    of the k-step, past the last sample) are fetched with an offset past the buffer descriptor's size
//    and arrive as zeros: the lane's offset holds the whole row, since the range check sees it alone.
//  * five LDS stages of 32 k rows.  In iteration i a wave waits for its
//    own loads of k-block i+1, meets the others at one barrier (which certifies block i+1 in
//    LDS and block i-1 no longer read), issues the loads of block i+4 into the stage block i-1
//    used, and computes block i.  A load has three iterations (about 3000 clocks) to land.
//    Operand fragments of the next k-step are fetched from LDS during the MFMAs of the current
//    one, across the barrier and across samples too, so the matrix pipe never waits for LDS latency.
//    The loads are issued from inline assembly because the compiler otherwise waits for every
//    outstanding LDS-DMA load before any LDS read; MFMAs, LDS reads and loads are interleaved by hand.
//  * per-sample weights: the accumulator holds sum_{j<=i} (w_j / w_i) G_j while sample i is added and is multiplied
//    by w_i / w_{i+1} at the boundary; samples of weight 0 are not read.  A sample takes ceil(T / 16) k-steps, two to a
//    k-block whatever samples they belong to, so no more than 15 rows a sample are padding (before: 31).
//    Weights are read 64 samples at a time, one a lane, and divided there; which of them count is a scalar mask: going
//    to the next sample is some scalar instructions and one lane read.  A scalar load of the weight and the division,
//    in the middle of the stream, cost more (~1200 clocks a sample) than the multiplies (~600, 128 a wave; the matrix
//    cores idle for most of them).  Blocks inside a sample test nothing of this, samples of one block each
//    (17 .. 32 tokens) next to nothing.  Gradient stage, us, before and after: 31 x 32 tokens, ten layers
//    704 x 704 37.6, 31.2; 64 x 32, eight layers 1024 wide 196, 161; 32 x 48 141, 118; 10 x 100, 24 layers 270, 246;
//    32 x 197, 48 layers 768 wide 1258, 1201; 4 x 2048, four layers 4096 wide 2872, 2854.
//    Few k-blocks are bound by what comes before and after them, so that the first weights are asked for before the tile is
//    located, the loads begin when it is known which samples count and the divisions wait until then (one sample: none),
//    and the last sample's blocks, of whatever number of k-steps, test nothing.  Gradient stage, us, on the 32-row blocks
//    with scalar loads, with all of it before the first load, and now: 64 tokens, eight layers 1024 wide 17.0, 17.8, 16.8;
//    16 tokens of 4096 170.8, 176.1, 167.7; 40 tokens, 24 layers 768 x 3072 82.0, 85.1, 82.7; two layers 3744 x 2352
//    32.6, 34.1, 32.9; 512 tokens, four layers 4096 wide 143.0, 146.2, 142.8.
//    Measured and not kept: multiplies between the matrix instructions, a branch or 16 multiplies for each (+9 % at 2048
//    tokens, no gain at 32); one of a SIMD's two waves multiplying after its block, the other before its
//    (64 x 32 tokens: 95 us where both before it take 87); all of the bookkeeping without branches (spills scalars).
#pragma once

#include <type_traits>

#include "dp_internal.h"
#include "lds_dma.h"

namespace dpbk {

template <int BM_, int WM_, int WN_, int NSTAGE_>
struct PipeShape {
  static constexpr int BM = BM_, BN = BM_, BK = 32, NSTAGE = NSTAGE_, WM = WM_, WN = WN_;
  static constexpr int NT = 64 * WM * WN;
  static constexpr int WTM = BM / WM, WTN = BN / WN;             // wave tile
  static constexpr int TM = WTM / 32, TN = WTN / 32;             // 32 x 32 MFMA tiles per wave
  static constexpr int ROW_BYTES = 2 * BM;
  static constexpr int TILE_BYTES = BK * ROW_BYTES;              // one operand, one stage
  static constexpr int STAGE_BYTES = 2 * TILE_BYTES;
  static constexpr int LDS_BYTES = NSTAGE * STAGE_BYTES;
  static constexpr int CHUNKS = BM / 8;                          // 16-byte chunks of a row
  static constexpr int ROWS_PER_LOAD = 64 / CHUNKS;              // of one wave
  static constexpr int LOADS = 2;                                // per operand, wave and k-block: 16 rows of the workgroup each
  static_assert(ROWS_PER_LOAD * WM * WN * LOADS == BK && TN == 2, "load split and fragment order");
};
using BigTile = PipeShape<256, 2, 4, 5>;
using MidTile = PipeShape<128, 2, 2, 5>;
using ShortTile = PipeShape<128, 2, 2, 3>;                         // 48 KiB: three workgroups per compute unit

// c *= f (the bits of a float) where turn is not zero.  Branch and multiplies are inside the assembly and every accumulator
// is one operand, so that for the compiler the contraction is one piece of straight code over whole register tuples:
// with multiplies, branches or second copies of the k-block of its own it moves the accumulators through scratch memory
// (126 to 540 registers) or through copies.  A tuple prints as v[first:last]; the inner loops read `first` off it.
// The compiler does not see into it, so the waits are counted here.  A vector instruction may touch the result of one of
// these matrix instructions (eight passes) after twelve others.  The multiplies go in the order of the matrix
// instructions: between the k-step's first one and the first multiply lie its other matrix instructions, its LDS reads and
// its loads (7 + 12 + 6 instructions of the 256 x 256 tile, 3 + 8 + 6 of the 128 x 128 one), and before the multiplies of
// the j-th accumulator 16 j others.  The s_nop is the wait of a matrix instruction for the last multiply.
#define DP_SCALE_TUPLES(tuples)                                                            \
  ".irp tuple, " tuples "\n\t"                                                             \
  ".set dp_first, 0\n\t"                                                                   \
  ".set dp_more, 1\n\t"                                                                    \
  ".irpc ch, \"\\tuple\"\n\t"                                                              \
  ".if '\\ch' == ':'\n\t.set dp_more, 0\n\t.endif\n\t"                                     \
  ".if dp_more && '\\ch' >= '0' && '\\ch' <= '9'\n\t"                                      \
  ".set dp_first, 10 * dp_first + ('\\ch' - '0')\n\t.endif\n\t"                            \
  ".endr\n\t"                                                                              \
  ".irp i, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15\n\t"                       \
  "v_mul_f32 v[dp_first+\\i], %[f], v[dp_first+\\i]\n\t"                                   \
  ".endr\n\t"                                                                              \
  ".endr\n\t"
__device__ __forceinline__ void scale_if(unsigned turn, unsigned f, f32x16 (&c)[4][2]) {
  asm volatile("s_cmp_eq_u32 %[turn], 0\n\ts_cbranch_scc1 .Lkeep%=\n\t"
               DP_SCALE_TUPLES("%0, %1, %2, %3, %4, %5, %6, %7") "s_nop 1\n.Lkeep%=:"
               : "+v"(c[0][0]), "+v"(c[0][1]), "+v"(c[1][0]), "+v"(c[1][1]), "+v"(c[2][0]), "+v"(c[2][1]), "+v"(c[3][0]),
                 "+v"(c[3][1])
               : [turn] "s"(turn), [f] "s"(f)
               : "scc");
}
__device__ __forceinline__ void scale_if(unsigned turn, unsigned f, f32x16 (&c)[2][2]) {
  asm volatile("s_cmp_eq_u32 %[turn], 0\n\ts_cbranch_scc1 .Lkeep%=\n\t"
               DP_SCALE_TUPLES("%0, %1, %2, %3") "s_nop 1\n.Lkeep%=:"
               : "+v"(c[0][0]), "+v"(c[0][1]), "+v"(c[1][0]), "+v"(c[1][1])
               : [turn] "s"(turn), [f] "s"(f)
               : "scc");
}
#undef DP_SCALE_TUPLES

// Weights of the samples window .. window + 63, one a lane; lanes from sample B on: not to be used.
__device__ __forceinline__ float window_weights(const float* C, unsigned window, int B) {
  const auto r = __builtin_amdgcn_make_buffer_rsrc((void*)(C + window), 0, 4 * min(B - (int)window, 64), 0x00020000);
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, 4 * (threadIdx.x & 63), 0, 0));
}

// Those of the first window by a load that the compiler leaves above what follows, branches too.
__device__ __forceinline__ float first_weights(const float* C, int B) {
  const float w = C[min(threadIdx.x & 63, (unsigned)B - 1)];
  asm volatile("" ::: "memory");
  return w;
}

// Samples [0, B) of the layer (one, `sample`, unless WEIGHTED) into `acc` (zeroed here); returns the weight the sum is
// expressed in (WEIGHTED; 0 when no sample counts), else 1.  C: weights by sample; w: those of the first window, which the
// caller asks for as early as it can (nothing is loaded before they are known).
template <class S, bool F16, bool WEIGHTED>
__device__ __forceinline__ float tn_contract(const void* a, const void* g, int T, int d, int p, int sample, int B,
                                             const float* C, float w, int m0, int n0, unsigned lds0,
                                             f32x16 (&acc)[S::TM][S::TN]) {
  constexpr int NSTAGE = S::NSTAGE, STAGE_BYTES = S::STAGE_BYTES, TILE_BYTES = S::TILE_BYTES, ROW_BYTES = S::ROW_BYTES;
  constexpr int BLOCK_LOADS = 2 * S::LOADS, KSTEP = 16;
  const int steps = (T + KSTEP - 1) / KSTEP;                      // of a sample
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform: keeps LDS bases scalar

  // ---- global -> LDS addressing: load ks of a wave covers rows ROWS_PER_LOAD wave + lane / CHUNKS of k-step ks of the
  // 32-row k-block; the lane's LDS chunk c holds logical chunk c ^ ((row & 3) << 2).
  const int lrow = wave * S::ROWS_PER_LOAD + lane / S::CHUNKS;
  const int chunk = (lane % S::CHUNKS) ^ ((lrow & 3) << 2);
  const unsigned a_org = m0 + chunk * 8 < d ? (unsigned)(lrow * d + m0 + chunk * 8) * 2u : OOB;
  const unsigned b_org = n0 + chunk * 8 < p ? (unsigned)(lrow * p + n0 + chunk * 8) * 2u : OOB;
  const unsigned a_slab = (unsigned)T * d * 2u, b_slab = (unsigned)T * p * 2u;
  const unsigned a_step = 2u * KSTEP * d, b_step = 2u * KSTEP * p;             // bytes of a k-step
  const unsigned lds_ld = lds0 + wave * 1024;
  // Prefetch stream: the next k-step to fetch lies va, vb (per lane) past the start of its sample, whose slabs ra and rb
  // describe; what lies past a descriptor's size arrives as zeros.  p_mask: the samples from this one on that count.
  // Past the last one the slabs are empty, and each k-step still issues the same number of loads.
  uint64_t p_mask = 1;
  i32x4 ra, rb;
  unsigned va, vb;
  int p_steps, p_stage;
  auto prefetch_a = [&](int ks) { load_to_lds(ra, va, 0, lds_ld + p_stage * STAGE_BYTES + ks * KSTEP * ROW_BYTES); };
  auto prefetch_b = [&](int ks) {
    load_to_lds(rb, vb, 0, lds_ld + p_stage * STAGE_BYTES + ks * KSTEP * ROW_BYTES + TILE_BYTES);
  };
  auto next_slab = [](i32x4& r, uint64_t bytes) {
    const uint64_t q = ((uint64_t)(uint32_t)r[1] << 32 | (uint32_t)r[0]) + bytes;
    r[0] = (int)(uint32_t)q;
    r[1] = (int)(uint32_t)(q >> 32);
  };
  auto prefetch_advance = [&](int ks) {
    va += a_step;
    vb += b_step;
    if (WEIGHTED && __builtin_expect(--p_steps == 0, 0)) {     // (one sample: the rows past its end are zeros anyway)
      p_steps = steps;
      va = a_org;
      vb = b_org;
      next_slab(ra, a_slab);
      next_slab(rb, b_slab);
      p_mask >>= 1;
      if ((p_mask & 1) == 0) {                         // the next sample does not count, or there is none
        if (p_mask == 0) {
          ra[2] = rb[2] = 0;
          p_steps = INT32_MAX;
        } else {
          const int n = __builtin_ctzll(p_mask);
          p_mask >>= n;
          next_slab(ra, (uint64_t)n * a_slab);
          next_slab(rb, (uint64_t)n * b_slab);
        }
      }
    }
    if (ks == 1) p_stage = p_stage + 1 == NSTAGE ? 0 : p_stage + 1;
  };

  // ---- LDS -> MFMA operand addressing ---------------------------------------------------
  // 16-lane block b = lane >> 4, s = lane & 15: row = 8*(b>>1) + (s>>2) (+4 for the second
  // half), element column = 16*(b&1) + 4*(s&3) inside a 32-wide MFMA tile.
  const int blk = lane >> 4, s = lane & 15;
  const int rrow = 8 * (blk >> 1) + (s >> 2);
  const int sw = (rrow & 3) << 2;
  const int wm = (wave / S::WN) * S::WTM, wn = (wave % S::WN) * S::WTN;
  unsigned a_rd[S::TM], b_rd[S::TN];
#pragma unroll
  for (int i = 0; i < S::TM; ++i) {
    const int ca = (wm + i * 32 + 16 * (blk & 1) + 4 * (s & 3)) >> 3;
    a_rd[i] = lds0 + rrow * ROW_BYTES + ((ca ^ sw) << 4) + (s & 1) * 8;
  }
#pragma unroll
  for (int i = 0; i < S::TN; ++i) {
    const int cb = (wn + i * 32 + 16 * (blk & 1) + 4 * (s & 3)) >> 3;
    b_rd[i] = lds0 + TILE_BYTES + rrow * ROW_BYTES + ((cb ^ sw) << 4) + (s & 1) * 8;
  }
#pragma unroll
  for (int x = 0; x < S::TM; ++x)
#pragma unroll
    for (int y = 0; y < S::TN; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
  // Fragments are read a k-step ahead, or a whole block (buffers of two blocks) where a wave's k-step is only 4
  // MFMAs, too short to cover the latency of the next one's reads, and the stream is one sample's:
  // 256 tiles of 128 x 128 over 2048 tokens 28.6 -> 25.0 us.  (Over weighted samples the two copies of
  // the block with the boundary test in front of each cost what the reads gain.)
  constexpr int DEPTH = !WEIGHTED && S::TM == 2 ? 2 : 1;
  Frag fa[2 * DEPTH][S::TM], fb[2 * DEPTH][S::TN];
  // Items 0 .. TM + 1 of a k-step's fragments in the order its matrix instructions need them.
  auto read_frag = [&](int buf, int q, int stage, int ks) {
    const bool is_b = q == 0 || q == 2;
    const int i = is_b ? q >> 1 : q == 1 ? 0 : q - 2;
    unsigned base = stage * STAGE_BYTES;
    asm("" : "+s"(base));                                // one address, the rest in the instructions' offsets
    const unsigned addr = (is_b ? b_rd[i] : a_rd[i]) + base + ks * KSTEP * ROW_BYTES;
    Frag& f = is_b ? fb[buf][i] : fa[buf][i];
    f.h[0] = lds_read_tr(addr);
    f.h[1] = lds_read_tr(addr + 4 * ROW_BYTES);
  };
  constexpr int ITEMS = S::TM + S::TN, STEPS = S::TM * S::TN;
  int c_stage;
  // The stream begins at sample smp: blocks 0 .. NSTAGE-2 in flight; then block 0 complete in LDS, its first fragments
  // requested.
  auto start_stream = [&](int smp) {
    c_stage = p_stage = 0;
    p_steps = steps;
    va = a_org;
    vb = b_org;
    ra = make_rsrc(static_cast<const unsigned char*>(a) + (size_t)smp * a_slab, a_slab);
    rb = make_rsrc(static_cast<const unsigned char*>(g) + (size_t)smp * b_slab, b_slab);
#pragma unroll 1
    for (int q = 0; q < NSTAGE - 1; ++q)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        prefetch_a(ks);
        prefetch_b(ks);
        prefetch_advance(ks);
      }
  };
  auto await_stream = [&]() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 2) * BLOCK_LOADS) : "memory");
    __syncthreads();
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
      read_frag(0, q, 0, 0);
      if (DEPTH == 2) read_frag(1, q, 0, 1);
    }
  };
  // A k-block: wait for block +1, barrier, two k-steps.
  auto open_block = [&]() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 3) * BLOCK_LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    DP_PIN();
  };
  // A k-step: STEPS MFMAs with the reads of the next fragments, one load of a and one of g of block +(NSTAGE-1) and the
  // scalar work of both streams (count: the compute stream's) between them.
  auto step = [&](auto ks_tag, auto parity_tag, auto next) {
    constexpr int ks = decltype(ks_tag)::value, parity = decltype(parity_tag)::value;
    const int n_stage = c_stage + 1 == NSTAGE ? 0 : c_stage + 1;
    // buffer in use; buffer, stage and k-step of the reads
    constexpr int use = 2 * parity + ks;
    constexpr int fill = DEPTH == 2 ? 2 * (parity ^ 1) + ks : ks ^ 1;
    const int r_stage = DEPTH == 1 && ks == 0 ? c_stage : n_stage;
    constexpr int r_ks = DEPTH == 2 ? ks : ks ^ 1;
#pragma unroll
    for (int slot = 0; slot < STEPS; ++slot) {
      const int x = slot / S::TN, y = slot % S::TN;
      acc[x][y] = mfma16<F16>(fb[use][y].v, fa[use][x].v, acc[x][y]);
      DP_PIN();
      if (slot < ITEMS) read_frag(fill, slot, r_stage, r_ks);
      constexpr int a_slot = STEPS == 8 ? 6 : 1, b_slot = STEPS - 1, next_slot = STEPS - 1;
      if (slot == a_slot) prefetch_a(ks);
      if (slot == b_slot) prefetch_b(ks);
      if (slot == next_slot) next(ks);
      DP_PIN();
    }
    if (ks == 1) c_stage = n_stage;
  };
  auto scale = [&](unsigned turn, unsigned f) {
    scale_if(turn, f, acc);
    DP_PIN();
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, 1> odd{};
  float held = 0.f;                                      // weight the accumulator is expressed in; 0: none yet
  if constexpr (WEIGHTED) {
    // Samples in windows of 64: their weights are in the lanes, which of them count in a scalar mask, so that the step
    // from one to the next is a few scalar instructions between matrix instructions.
    for (unsigned window = 0; window < (unsigned)B; window += 64) {
      if (window > 0) w = window_weights(C, window, B);
      uint64_t mask = __ballot(w != 0.f && window + lane < (unsigned)B);
      if (mask == 0) continue;
      if (held != 0.f) __syncthreads();                  // the last window's fragments are read
      const int first = __builtin_ctzll(mask);
      const uint64_t p_all = mask >> first;
      p_mask = p_all;
      start_stream(window + first);                      // the ratios while its first loads are on their way
      float ratio = 1.f;
      if (B > 1) {                                       // one sample: nothing to go on from
        const uint64_t before = mask & ((1ull << lane) - 1);
        const float prev = __shfl(w, before ? 63 - __builtin_clzll(before) : lane);
        ratio = before ? prev / w : held != 0.f ? held / w : 1.f;
      }
      held = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), 63 - __builtin_clzll(mask)));
      await_stream();
      constexpr unsigned kOne = 0x3f800000u;             // bits of 1.f
      int n = __builtin_popcountll(mask) * steps;        // odd: the last k-step's rows are zeros
      // f: ratio of the sample that comes next; turn: not zero where the next k-step is its first and it is not 1
      unsigned f = __builtin_amdgcn_readlane(__float_as_uint(ratio), first), turn = f ^ kOne;
      int left;                                          // k-steps to the end of the sample at hand; two more for the last one
      unsigned f_next;                                   // the ratio of the sample after the one at hand
      auto to_next = [&]() {
        mask &= mask - 1;
        f_next = mask ? __builtin_amdgcn_readlane(__float_as_uint(ratio), __builtin_ctzll(mask)) : kOne;
        left = mask ? steps : steps + 2;
      };
      to_next();
      auto count = [&](int ks) {
        prefetch_advance(ks);
        f = f_next;
        turn = 0;
        if (--left == 0) {
          turn = f_next ^ kOne;
          to_next();
        }
      };
      if (steps == 2 && (p_all & (p_all + 1)) == 0) {
        // Samples of one block each, all of which count: nothing to test but the end.
        int p_samples = __builtin_popcountll(p_mask), j = first + 1;
        const int end = first + n / 2;
        auto next = [&](int ks) {
          if (ks == 0) {
            va += a_step;
            vb += b_step;
            return;
          }
          va = a_org;
          vb = b_org;
          next_slab(ra, a_slab);
          next_slab(rb, b_slab);
          --p_samples;
          ra[2] = p_samples > 0 ? (int)a_slab : 0;
          rb[2] = p_samples > 0 ? (int)b_slab : 0;
          p_stage = p_stage + 1 == NSTAGE ? 0 : p_stage + 1;
          f = j < end ? __builtin_amdgcn_readlane(__float_as_uint(ratio), j & 63) : kOne;
        };
        do {
          open_block();
          scale(f ^ kOne, f);
          step(even, even, next);
          step(odd, even, next);
        } while (j++ < end);
        n = 0;
      }
      while (n > 0) {
        if (turn == 0) {
          for (; left > 2; left -= 2, n -= 2) {          // blocks inside the sample, or to the end of the last one
            open_block();
            step(even, even, prefetch_advance);
            step(odd, even, prefetch_advance);
          }
          if (n <= 0) break;
        }
        n -= 2;
        open_block();
        scale(turn, f);
        step(even, even, count);
        scale(turn, f);
        step(odd, even, count);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // zero-fill loads past the end
    }
  } else {                                               // one sample
    held = 1.f;
    start_stream(sample);
    await_stream();
    const int nkb = (T + S::BK - 1) / S::BK;
    for (int kb = 0; kb < nkb; kb += DEPTH) {
      open_block();
      step(even, even, prefetch_advance);
      step(odd, even, prefetch_advance);
      if (DEPTH == 2 && kb + 1 < nkb) {
        constexpr std::integral_constant<int, DEPTH - 1> second{};
        open_block();
        step(even, second, prefetch_advance);
        step(odd, second, prefetch_advance);
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // zero-fill loads past the end
  }
  return held;
}

}  // namespace dpbk
