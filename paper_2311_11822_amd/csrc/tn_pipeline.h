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
//    against ~1400 per 32 tokens, here ~900.  Eight 1024-wide layers (gradient stage): 64 x 64 tokens 410 ->
//    268 us, 32 x 128 316 -> 240; 12 GPT blocks of width 768, 16 x 256 tokens 780 -> 704, of 1280, 8 x 512
//    1863 -> 1787; at 2048 tokens 3 % faster.
//  * global -> LDS without passing through registers (buffer_load ... lds, 16 B per lane).
//    A wave's load lands as 1 KiB of consecutive LDS = two 512-byte (four 256-byte) k rows, so rows cannot be
//    padded; instead the 16-byte chunks of row k are XOR-swizzled by (k & 3) << 2, which
//    spreads four consecutive k rows over the four 64-byte bank groups the transposing read
//    touches at once.  Out-of-range chunks (tile edge, rows past the end of a sample whose T is no multiple
//    of the k-block, past the last k-block) are fetched with an offset past the buffer descriptor's size
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
//    by w_i / w_{i+1} at the boundary; samples of weight 0 are not read.  Folding the
//    multiplies into the boundary block's MFMA stream needs a second copy of the block, between which the
//    compiler moves the accumulators through scratch memory (126 registers spilled).
#pragma once

#include <type_traits>

#include "dp_internal.h"
#include "lds_dma.h"

namespace dpbk {

template <int BM_, int WM_, int WN_>
struct PipeShape {
  static constexpr int BM = BM_, BN = BM_, BK = 32, NSTAGE = 5, WM = WM_, WN = WN_;
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
using BigTile = PipeShape<256, 2, 4>;
using MidTile = PipeShape<128, 2, 2>;

typedef const __attribute__((address_space(4))) float* const_floats;

// Samples [first, end) of the layer (one, unless WEIGHTED) into `acc` (zeroed here); returns the weight the sum is
// expressed in (WEIGHTED; 0 when no sample counts), else 1.  C: weights by sample, read by scalar loads (a vector load
// would make the compiler wait for every outstanding prefetch load).
template <class S, bool F16, bool WEIGHTED>
__device__ __forceinline__ float tn_contract(const void* a, const void* g, int T, int d, int p, int first_sample,
                                             int end_sample, const_floats C, int m0, int n0, unsigned lds0,
                                             f32x16 (&acc)[S::TM][S::TN]) {
  constexpr int NSTAGE = S::NSTAGE, STAGE_BYTES = S::STAGE_BYTES, TILE_BYTES = S::TILE_BYTES, ROW_BYTES = S::ROW_BYTES;
  constexpr int BLOCK_LOADS = 2 * S::LOADS;
  const int nkb = (T + S::BK - 1) / S::BK;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform: keeps LDS bases scalar

  // ---- global -> LDS addressing: load j of a wave covers rows 16 j + ROWS_PER_LOAD wave + lane / CHUNKS of
  // the 32-row k-block; the lane's LDS chunk c holds logical chunk c ^ ((row & 3) << 2).
  const int lrow = wave * S::ROWS_PER_LOAD + lane / S::CHUNKS;
  const int chunk = (lane % S::CHUNKS) ^ ((lrow & 3) << 2);
  const unsigned a_org = m0 + chunk * 8 < d ? (unsigned)(lrow * d + m0 + chunk * 8) * 2u : OOB;
  const unsigned b_org = n0 + chunk * 8 < p ? (unsigned)(lrow * p + n0 + chunk * 8) * 2u : OOB;
  const unsigned a_half = 16u * d * 2u, b_half = 16u * p * 2u;       // bytes per 16 rows
  const unsigned a_slab = (unsigned)T * d * 2u, b_slab = (unsigned)T * p * 2u;
  const unsigned char* a_base = static_cast<const unsigned char*>(a);
  const unsigned char* b_base = static_cast<const unsigned char*>(g);
  const unsigned lds_ld = lds0 + wave * 1024;
  auto skip = [&](int i) {                             // first sample from i on that counts
    if (WEIGHTED)
      while (i < end_sample && C[i] == 0.f) ++i;
    return i;
  };
  // Prefetch stream: (p_i, p_kb) is the next k-block to fetch.  Once p_i >= end_sample ("past the
  // end") every lane fetches zeros, so each iteration issues the same number of loads.
  int p_i = skip(first_sample), p_kb = 0, p_stage = 0;
  i32x4 ra, rb;
  unsigned va, vb;                 // per-lane byte offset of the k-block's row inside the slab, or past OOB
  auto prefetch_sample = [&]() {
    const bool valid = p_i < end_sample;
    const int smp = valid ? p_i : first_sample;
    ra = make_rsrc(a_base + (size_t)smp * a_slab, a_slab);
    rb = make_rsrc(b_base + (size_t)smp * b_slab, b_slab);
    va = valid ? a_org : OOB;
    vb = valid ? b_org : OOB;
  };
  prefetch_sample();
  auto prefetch_issue = [&](int x) {                   // x = 0, 1: a; 2, 3: g
    const unsigned dst = lds_ld + p_stage * STAGE_BYTES + (x & 1) * 16 * ROW_BYTES;
    if (x < 2)
      load_to_lds(ra, va + (x & 1) * a_half, 0, dst);
    else
      load_to_lds(rb, vb + (x & 1) * b_half, 0, dst + TILE_BYTES);
  };
  auto prefetch_advance = [&]() {
    va += 2 * a_half;
    vb += 2 * b_half;
    if (WEIGHTED && p_i < end_sample && ++p_kb == nkb) {       // (one sample: the rows past its end are zeros anyway)
      p_kb = 0;
      p_i = skip(p_i + 1);
      prefetch_sample();
    }
    p_stage = p_stage + 1 == NSTAGE ? 0 : p_stage + 1;
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
    const unsigned o = stage * STAGE_BYTES + ks * 16 * ROW_BYTES;
    if (q == 0 || q == 2) {
      fb[buf][q >> 1].h[0] = lds_read_tr(b_rd[q >> 1] + o);
      fb[buf][q >> 1].h[1] = lds_read_tr(b_rd[q >> 1] + o + 4 * ROW_BYTES);
    } else {
      const int i = q == 1 ? 0 : q - 2;
      fa[buf][i].h[0] = lds_read_tr(a_rd[i] + o);
      fa[buf][i].h[1] = lds_read_tr(a_rd[i] + o + 4 * ROW_BYTES);
    }
  };

  // Compute stream over the samples that count.
  int c_i = p_i;
  if (c_i >= end_sample) return 0.f;
  float held = WEIGHTED ? C[c_i] : 1.f;
  // prologue: blocks 0 .. NSTAGE-2 in flight; block 0 complete in LDS
  for (int q = 0; q < NSTAGE - 1; ++q) {
#pragma unroll
    for (int x = 0; x < BLOCK_LOADS; ++x) prefetch_issue(x);
    prefetch_advance();
  }
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 2) * BLOCK_LOADS) : "memory");
  __syncthreads();
  constexpr int ITEMS = S::TM + S::TN, STEPS = S::TM * S::TN;
#pragma unroll
  for (int q = 0; q < ITEMS; ++q) {
    read_frag(0, q, 0, 0);
    if (DEPTH == 2) read_frag(1, q, 0, 1);
  }

  int c_stage = 0;
  // One k-block: wait for block +1, barrier, 2 STEPS MFMAs with the reads of the next fragments and the
  // loads of block +(NSTAGE-1) between them.
  auto block = [&](auto parity_tag) {
    constexpr int parity = decltype(parity_tag)::value;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 3) * BLOCK_LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    const int n_stage = c_stage + 1 == NSTAGE ? 0 : c_stage + 1;
    DP_PIN();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      // buffer in use; buffer, stage and k-step of the reads
      const int use = 2 * parity + ks;
      const int fill = DEPTH == 2 ? 2 * (parity ^ 1) + ks : ks ^ 1;
      const int r_stage = DEPTH == 1 && ks == 0 ? c_stage : n_stage, r_ks = DEPTH == 2 ? ks : ks ^ 1;
#pragma unroll
      for (int x = 0; x < S::TM; ++x)
#pragma unroll
        for (int y = 0; y < S::TN; ++y) {
          acc[x][y] = mfma16<F16>(fb[use][y].v, fa[use][x].v, acc[x][y]);
          DP_PIN();
          const int slot = S::TN * x + y;
          if (slot < ITEMS) read_frag(fill, slot, r_stage, r_ks);
          // one load of a (item ks) and one of g (2 + ks) per k-step
          constexpr int a_slot = STEPS == 8 ? 6 : 1, b_slot = STEPS - 1;
          if (slot == a_slot) prefetch_issue(ks);
          if (slot == b_slot) prefetch_issue(2 + ks);
          DP_PIN();
        }
    }
    prefetch_advance();
    c_stage = n_stage;
  };
  constexpr std::integral_constant<int, 0> even{};
  constexpr std::integral_constant<int, DEPTH - 1> odd{};
  if constexpr (WEIGHTED) {
    bool first = true;
    while (c_i < end_sample) {
      const float c = C[c_i];
      const float f = first ? 1.f : held / c;            // re-express the accumulator in this sample's weight
      first = false;
      held = c;
      if (f != 1.f)
#pragma unroll
        for (int x = 0; x < S::TM; ++x)
#pragma unroll
          for (int y = 0; y < S::TN; ++y)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[x][y][r] *= f;
      for (int kb = 0; kb < nkb; ++kb) block(even);
      c_i = skip(c_i + 1);
    }
  } else {                                               // one sample
    for (int kb = 0; kb < nkb; kb += DEPTH) {
      block(even);
      if (DEPTH == 2 && kb + 1 < nkb) block(odd);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // zero-fill loads past the end
  return held;
}

}  // namespace dpbk
