// Clip-weighted token contraction of whole 32-row k-blocks, tile after tile:
//   acc[j,k] = sum_i w_i sum_t a[i,t,j] g[i,t,k].
//
// The data path is that of tn_pipeline.h (global -> LDS directly, transposing LDS reads, a ring of k-blocks, one barrier a
// k-block, fragments read ahead); what differs:
//  * Under load the card is held by its power: the 32x32x16 loop runs at 1.56 to 1.7 GHz on real data.  16x16x32 matrix
//    instructions move half as many accumulator bytes a multiply-add: on random data in registers they reach 1.94 to 2.07
//    PFLOP/s where 32x32x16 ones reach 1.74 to 1.84.  A loop of them takes more clocks a k-block (1400 and 1290, the matrix
//    instructions alone 1056 and 1037: each holds the wave's issue port for 8 clocks, and the 96 KiB that LDS returns
//    hold the register ports for some 190) at 1.85 instead of 1.68 GHz.  Gradients, us, 32x32x16 and this: 4 x 2048 tokens,
//    12288 x 12288 1964, 1902; 4 x 1024, 12 layers of GPT width 2048 1111, 1065; 8 x 512, 48 of width 1280 1743, 1672;
//    16 x 256, 48 of width 768 676, 650; 64 x 64, eight 1024 x 1024 89, 81.  The order of the additions is that of two
//    32x32x16 steps: the same bits.
//  * A sample takes whole k-blocks, so that up to 31 rows a sample are zeros; where that costs more than the above gains,
//    the 16-row steps of tn_pipeline.h are used (whole_blocks in grad_gemm.hip).
//  * 256 workgroups go from tile to tile: the stream of k-blocks runs on into the next tile while the last one's sums go out
//    through the one stage that is free then, so that neither the launch of a workgroup nor its first loads are waited for.
//    The stores' way to memory (67 MB a round of 256 tiles, some 10 us) runs beside the next tile's first k-blocks.
//    48 layers of width 768, 16 x 256 tokens 658, 650; of width 1280, 8 x 512 1695, 1672; 32 x 64 380, 374.
//  * On 256 x 256 tiles one wave of a SIMD's two goes before the other (s_setprio): 0.5 to 1.5 %.  (On 128 x 128 ones a SIMD's waves
//    are of different workgroups and each workgroup waits for its last: 64 tokens, 20 layers of width 896 21.1 us, with it 24.6.)
//  * A new sample's first k-block multiplies each accumulator by the ratio of the weights two matrix instructions ahead of its use
//    (some 700 clocks a sample; all of them ahead of the k-block 1000).
#pragma once

#include <type_traits>

#include "dp_internal.h"
#include "lds_dma.h"
#include "tn_pipeline.h"

namespace dpbk {

// c *= f (the bits of a float).  Inside the assembly the accumulator stays one operand: with multiplies of its own the
// compiler moves accumulators through copies.  A tuple prints as v[first:last]; the inner loop reads `first` off it.
// The compiler does not see into it, so the waits are counted here: a vector instruction may touch the result of one
// of these matrix instructions (four passes) after eight others, and a matrix instruction that of a multiply after two.
__device__ __forceinline__ void scale_tuple(f32x4& c, unsigned f) {
  asm volatile(
      ".set dp_first, 0\n\t"
      ".set dp_more, 1\n\t"
      ".irpc ch, \"%0\"\n\t"
      ".if '\\ch' == ':'\n\t.set dp_more, 0\n\t.endif\n\t"
      ".if dp_more && '\\ch' >= '0' && '\\ch' <= '9'\n\t"
      ".set dp_first, 10 * dp_first + ('\\ch' - '0')\n\t.endif\n\t"
      ".endr\n\t"
      "v_mul_f32 v[dp_first], %1, v[dp_first]\n\t"
      "v_mul_f32 v[dp_first+1], %1, v[dp_first+1]\n\t"
      "v_mul_f32 v[dp_first+2], %1, v[dp_first+2]\n\t"
      "v_mul_f32 v[dp_first+3], %1, v[dp_first+3]"
      : "+v"(c)
      : "s"(f));
}

struct WeightedTile {
  int l, m0, n0;                                         // layer, origin
};

// Tiles id, id + stride, ... below end: contraction, then finish(tile, sums, the weight they are in, the wave's LDS, its place
// in the tile, what to call ahead of the first store).  locate.tile(id): the tile's number as the layers count them;
// locate(ga, tile, id): its origin, false where it lies past the layer's edge.  More than one tile to a workgroup (CHAIN): all layers
// of one T, and no more than 64 samples.
template <class S, bool F16, bool CHAIN, class Locate, class Finish>
__device__ __forceinline__ void weighted_tiles(const GroupArgs& ga, const float* C_all, int id, int stride, int end,
                                               Locate locate, Finish finish) {
  constexpr int NSTAGE = S::NSTAGE, STAGE_BYTES = S::STAGE_BYTES, TILE_BYTES = S::TILE_BYTES, ROW_BYTES = S::ROW_BYTES;
  constexpr int BLOCK_LOADS = 2 * S::LOADS, HALF = 16;
  constexpr int XM = S::WTM / 16, XN = S::WTN / 16, GX = XM / 2, SLOTS = GX * XN;     // 16 x 16 tiles of a wave; of half a k-block
  static_assert(XN == 4 && (XM == 4 || XM == 8), "order of the operands' reads");
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds_raw[];
  const unsigned lds0 = (unsigned)(uintptr_t)lds_raw;
  const int B = ga.B;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);         // wave-uniform: keeps LDS bases scalar

  // The layers' first tiles, one a lane, for all lookups of this wave.
  const int begin = lane < ga.n_layers ? ga.layer[lane < ga.n_layers ? lane : 0].tile_begin : INT32_MAX;
  auto layer_at = [&](int tile) { return __builtin_popcountll(__ballot(begin <= tile)) - 1; };
  auto weights_at = [&](int l) { return window_weights(C_all + ga.layer[l].c_off, 0, B); };
  WeightedTile cur = {layer_at(locate.tile(id)), 0, 0};
  float w = weights_at(cur.l), w_next = 0.f;
  if (CHAIN && id + stride < end) w_next = weights_at(layer_at(locate.tile(id + stride)));
  if (!locate(ga, cur, id)) return;
  const int blocks = (ga.layer[cur.l].T + S::BK - 1) / S::BK;        // of a sample

  // ---- global -> LDS: load h of a wave covers rows ROWS_PER_LOAD wave + lane / CHUNKS of half h of the k-block; the lane's LDS
  // chunk c holds logical chunk c ^ (4 (row & 3) + 2 (row >> 3 & 1)): the transposing read takes four rows of 32 bytes
  // from rows r .. r + 3 and from eight rows below at once, which lie in eight different 32-byte bank groups so.
  const int lrow = wave * S::ROWS_PER_LOAD + lane / S::CHUNKS;
  const int chunk = (lane % S::CHUNKS) ^ ((lrow & 3) << 2 | (lrow >> 3 & 1) << 1);
  const unsigned lds_ld = lds0 + wave * 1024;
  // The stream of k-blocks: the next half to fetch lies va, vb (per lane) past the start of its sample, whose slabs ra and rb
  // describe; what lies past a descriptor's size arrives as zeros.  p_mask: the samples from this one on that count.
  unsigned a_org, b_org, a_slab, b_slab, a_step, b_step, va, vb;
  uint64_t p_mask = 1;
  i32x4 ra, rb;
  int p_left, p_stage;
  auto open_stream = [&](const WeightedTile& t, int smp) {
    const GroupLayer& ly = ga.layer[t.l];
    const int d = ly.d_in, p = ly.d_out;
    a_slab = (unsigned)ly.T * d * 2u;
    b_slab = (unsigned)ly.T * p * 2u;
    a_step = 2u * HALF * d;
    b_step = 2u * HALF * p;
    a_org = t.m0 + chunk * 8 < d ? (unsigned)(lrow * d + t.m0 + chunk * 8) * 2u : OOB;
    b_org = t.n0 + chunk * 8 < p ? (unsigned)(lrow * p + t.n0 + chunk * 8) * 2u : OOB;
    va = a_org;
    vb = b_org;
    p_left = blocks;
    ra = make_rsrc(static_cast<const unsigned char*>(ly.a) + (size_t)smp * a_slab, a_slab);
    rb = make_rsrc(static_cast<const unsigned char*>(ly.g) + (size_t)smp * b_slab, b_slab);
  };
  auto prefetch_a = [&](int h) {
    load_to_lds(ra, va, 0, lds_ld + p_stage * STAGE_BYTES + h * HALF * ROW_BYTES);
    va += a_step;
  };
  auto prefetch_b = [&](int h) {
    load_to_lds(rb, vb, 0, lds_ld + p_stage * STAGE_BYTES + h * HALF * ROW_BYTES + TILE_BYTES);
    vb += b_step;
  };
  auto next_slab = [](i32x4& r, uint64_t bytes) {
    const uint64_t q = ((uint64_t)(uint32_t)r[1] << 32 | (uint32_t)r[0]) + bytes;
    r[0] = (int)(uint32_t)q;
    r[1] = (int)(uint32_t)(q >> 32);
  };
  WeightedTile nxt = cur;
  uint64_t mask_next = 0;                                // samples of tile nxt that count
  bool chain = false;                                    // the stream goes on with tile nxt
  auto prefetch_advance = [&]() {
    p_stage = p_stage + 1 == NSTAGE ? 0 : p_stage + 1;
    if (__builtin_expect(--p_left == 0, 0)) {
      p_left = blocks;
      va = a_org;
      vb = b_org;
      next_slab(ra, a_slab);
      next_slab(rb, b_slab);
      p_mask >>= 1;
      if ((p_mask & 1) == 0) {                           // the next sample does not count, or there is none
        if (p_mask == 0) {
          if (CHAIN && chain) {
            const int first = __builtin_ctzll(mask_next);
            p_mask = mask_next >> first;
            open_stream(nxt, first);
          } else {                                       // zeros from here on, the same number of loads
            ra[2] = rb[2] = 0;
            p_left = INT32_MAX;
          }
        } else {
          const int n = __builtin_ctzll(p_mask);
          p_mask >>= n;
          next_slab(ra, (uint64_t)n * a_slab);
          next_slab(rb, (uint64_t)n * b_slab);
        }
      }
    }
  };

  // ---- LDS -> MFMA operands: lanes 16 b .. 16 b + 15 hold rows 8 b .. 8 b + 7 of 16 columns; the lane's address of the read is
  // row 8 b + (s >> 2) (+ 4 for the second half), columns 4 (s & 3) of them.
  const int s = lane & 15;
  const int rrow = 8 * (lane >> 4) + (s >> 2);
  const int sw = (rrow & 3) << 2 | (rrow >> 3 & 1) << 1;
  const int wm = (wave / S::WN) * S::WTM, wn = (wave % S::WN) * S::WTN;
  const unsigned a_rd = lds0 + rrow * ROW_BYTES + ((((wm + 4 * (s & 3)) >> 3) ^ sw) << 4) + (s & 1) * 8;
  const unsigned b_rd = lds0 + TILE_BYTES + rrow * ROW_BYTES + ((((wn + 4 * (s & 3)) >> 3) ^ sw) << 4) + (s & 1) * 8;
  f32x4 acc[XM][XN];
  Frag fa[XM], fb[XN];
  auto read_frag = [&](Frag& f, unsigned rd, int i, int stage) {
    unsigned base = stage * STAGE_BYTES;
    asm("" : "+s"(base));                                // one address, the rest in the instructions' offsets
    const unsigned addr = (rd ^ (unsigned)(i << 5)) + base;
    f.h[0] = lds_read_tr(addr);
    f.h[1] = lds_read_tr(addr + 4 * ROW_BYTES);
  };
  int c_stage = 0;
  auto first_frags = [&]() {
#pragma unroll
    for (int q = 0; q < GX; ++q) read_frag(fa[q], a_rd, q, c_stage);
#pragma unroll
    for (int q = 0; q < XN - 1; ++q) read_frag(fb[q], b_rd, q, c_stage);
  };
  // Wait for block +1, barrier.
  auto open_block = [&]() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 3) * BLOCK_LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    DP_PIN();
  };
  // A k-block: two halves of the a operands, in each g outside a, so that an operand's registers are free SLOTS or more matrix
  // instructions before they are needed again: all operands are read a dozen instructions ahead without a second set
  // of registers.  Between them one load of a and of g of block +(NSTAGE - 1) a half.  SCALED: of a new sample, accumulators times f.
  auto block = [&](auto scaled, unsigned f, auto next) {
    constexpr bool SCALED = decltype(scaled)::value;
    const int n_stage = c_stage + 1 == NSTAGE ? 0 : c_stage + 1;
    auto scale = [&](int q) { scale_tuple(acc[GX * (q / SLOTS) + q % SLOTS % GX][q % SLOTS / GX], f); };
    if constexpr (SCALED) {
      scale(0);
      scale(1);
      DP_PIN();
    }
#pragma unroll
    for (int half = 0; half < 2; ++half)
#pragma unroll
      for (int slot = 0; slot < SLOTS; ++slot) {
        const int x0 = slot % GX, x = GX * half + x0, y = slot / GX;
        acc[x][y] = mfma16<F16>(fb[y].v, fa[x].v, acc[x][y]);
        DP_PIN();
        if constexpr (SCALED) {
          const int q = SLOTS * half + slot + 2;         // the last one beside the one before it: no multiplies come between later
          if (q < 2 * SLOTS - 1) scale(q);
          if (q == 2 * SLOTS - 2) scale(q + 1);
        }
        if (half == 0) {
          constexpr int EVERY = GX == 4 ? 3 : 1;
          if (slot == 0) read_frag(fb[XN - 1], b_rd, XN - 1, c_stage);
          if (slot > 0 && (slot - 1) % EVERY == 0 && (slot - 1) / EVERY < GX)
            read_frag(fa[GX + (slot - 1) / EVERY], a_rd, GX + (slot - 1) / EVERY, c_stage);
        } else {
          if (slot < GX) read_frag(fa[slot], a_rd, slot, n_stage);
          if (slot > 0 && x0 == 0) read_frag(fb[y - 1], b_rd, y - 1, n_stage);
        }
        constexpr int A_SLOT = GX == 4 ? 6 : 3, B_SLOT = GX == 4 ? 11 : 5;
        if (slot == A_SLOT) prefetch_a(half);
        if (slot == B_SLOT) prefetch_b(half);
        if (half == 1 && slot == SLOTS - 1) next();
        DP_PIN();
      }
    c_stage = n_stage;
  };
  constexpr std::true_type rescaled{};
  constexpr std::false_type plain{};
  constexpr unsigned kOne = 0x3f800000u;                 // bits of 1.f
  if (S::NT == 512 && wave < 4) __builtin_amdgcn_s_setprio(3);
  // joined: the stream was opened by the tile before, NSTAGE - 1 blocks of it are in LDS.
  bool joined = false, dirty = false;
#pragma unroll 1
  for (;;) {
    const bool more = CHAIN && id + stride < end;
    if (more) {
      nxt.l = layer_at(locate.tile(id + stride));
      locate(ga, nxt, id + stride);
      mask_next = __ballot(w_next != 0.f && lane < B);
    }
#pragma unroll
    for (int x = 0; x < XM; ++x)
#pragma unroll
      for (int y = 0; y < XN; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[x][y][r] = 0.f;
    float held = 0.f;                                    // weight the accumulator is expressed in; 0: none yet
    chain = false;
    // Samples in windows of 64: their weights are in the lanes, which of them count in a scalar mask.
#pragma unroll 1
    for (unsigned window = 0; window < (unsigned)B; window += 64) {
      if (window > 0) w = window_weights(C_all + ga.layer[cur.l].c_off, window, B);
      const uint64_t mask = __ballot(w != 0.f && window + lane < (unsigned)B);
      if (mask == 0) continue;
      const int first = __builtin_ctzll(mask);
      // Tiles of fewer blocks than the ring has are not joined: the stream would run through them into a third tile.
      if (CHAIN)
        chain = more && __builtin_popcountll(mask) * blocks >= NSTAGE && __builtin_popcountll(mask_next) * blocks >= NSTAGE;
      if (!joined) {
        if (dirty || held != 0.f) __syncthreads();       // the last fragments, or rows on their way out, are read
        p_mask = mask >> first;
        p_stage = c_stage = 0;
        open_stream(cur, window + first);                // the ratios while its first loads are on their way
#pragma unroll 1
        for (int q = 0; q < NSTAGE - 1; ++q) {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            prefetch_a(h);
            prefetch_b(h);
          }
          prefetch_advance();
        }
      }
      float ratio = 1.f;
      if (B > 1) {                                       // one sample: nothing to go on from
        const uint64_t before = mask & ((1ull << lane) - 1);
        const float prev = __shfl(w, before ? 63 - __builtin_clzll(before) : lane);
        ratio = before ? prev / w : held != 0.f ? held / w : 1.f;
      }
      held = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), 63 - __builtin_clzll(mask)));
      // Runs of samples of one weight: where they begin, and the ratio and the k-blocks of the one that comes next.
      uint64_t heads = mask & (__ballot(ratio != 1.f) | 1ull << first);
      unsigned f;
      int left = 0, left_next;
      auto look_ahead = [&]() {
        const uint64_t rest = heads & (heads - 1), before = (heads & -heads) - 1, until = rest ? (rest & -rest) - 1 : ~0ull;
        f = heads ? __builtin_amdgcn_readlane(__float_as_uint(ratio), __builtin_ctzll(heads)) : kOne;
        left_next = heads ? __builtin_popcountll(mask & until & ~before) * blocks : 0;
        heads = rest;
      };
      look_ahead();
      if (!joined) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTAGE - 2) * BLOCK_LOADS) : "memory");
        __syncthreads();
      }
      first_frags();
      if (CHAIN && joined) {
        // Blocks 1 .. NSTAGE - 2 are in LDS, certified by these barriers: a wait would be one for the last tile's stores.
#pragma unroll 1
        for (int q = 0; q < NSTAGE - 2; ++q) {
          __builtin_amdgcn_s_barrier();
          DP_PIN();
          const bool head = left == 0;
          block(rescaled, head ? f : kOne, [&]() {
            prefetch_advance();
            if (head) {
              left = left_next;
              look_ahead();
            }
            --left;
          });
        }
        for (; left > 0; --left) {
          open_block();
          block(plain, kOne, prefetch_advance);
        }
      }
      while (left_next) {
        open_block();
        block(rescaled, f, [&]() {
          prefetch_advance();
          left = left_next;
          look_ahead();
        });
        for (--left; left > 0; --left) {
          open_block();
          block(plain, kOne, prefetch_advance);
        }
      }
      if (!chain) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // zero-fill loads past the end
    }
    if (CHAIN && id + 2 * stride < end) w = weights_at(layer_at(locate.tile(id + 2 * stride)));
    __syncthreads();                                     // the last block's stage is read
    finish(cur, acc, held, lds0 + (c_stage == 0 ? NSTAGE - 1 : c_stage - 1) * STAGE_BYTES + wave * (STAGE_BYTES / (S::WM * S::WN)),
           wm, wn, [&]() { asm volatile("s_waitcnt vmcnt(0)" : "+v"(w) : : "memory"); });   // the joined stream's first blocks
    if (!more) return;
    const float t = w;
    w = w_next;
    w_next = t;
    cur = nxt;
    id += stride;
    joined = chain;
    dirty = true;
  }
}

// The same contraction on a 64 x 64 tile, four waves of 32 x 32, for the few tiles at the end of a launch: a wave has four
// matrix instructions (64 clocks) a k-block, so what counts is what lies between them: two k-blocks to a barrier, four sets of
// fragments, the next two blocks' read during these two's matrix instructions, the samples' bookkeeping in scalars beside
// them; a ring of ten 8 KiB stages with eight blocks on their way (sixteen stages: no faster).  A block takes some 370 clocks, 49
// instructions of each wave.  Gradients, us, through registers with 64-row blocks and a barrier each, with one block to a barrier here,
// and now: 16 x 256 tokens, one layer 1024 x 1024 29.6, 26.6, 25.1; two 39.1, 33.0, 32.4; 32 x 197, three 768 x 768 68.8, 52.0,
// 50.1; 32 x 64, two 1024 x 1024 30.3, 23.9, 22.7; 64 x 32, one 49.6, 24.3, 23.0; 4 x 256, two 512 x 512 10.9, 10.4, 10.0.
struct SmallTile {
  static constexpr int BM = 64, BK = 32, NSTAGE = 10, NT = 256;
  static constexpr int ROW_BYTES = 2 * BM, TILE_BYTES = BK * ROW_BYTES, STAGE_BYTES = 2 * TILE_BYTES;
  static constexpr int LDS_BYTES = NSTAGE * STAGE_BYTES;            // 80 KiB: two workgroups per compute unit
};

// The four accumulators times f (the bits of a float) where turn is not zero; waits as at scale_tuple.  The matrix instructions go
// c00, c10, c01, c11, the multiplies c00, c01, c10, c11, four each, behind a compare and a branch.  Between a k-block's c01 and its
// multiplies lie c11, four LDS reads, the scalars, compare and branch, and four multiplies; between c11 and its own two LDS
// reads, the same scalars and branch and twelve multiplies: more than eight, with the pair's barrier between (its first k-block)
// or without (its second).  Between the last multiply, of c11, and c11's matrix instruction lie the s_nop and three others; before
// c00's the multiplies of the other three.
__device__ __forceinline__ void scale_if(unsigned turn, unsigned f, f32x4 (&c)[2][2]) {
  asm volatile(
      "s_cmp_eq_u32 %[turn], 0\n\ts_cbranch_scc1 .Lkeep%=\n\t"
      ".irp tuple, %0, %1, %2, %3\n\t"
      ".set dp_first, 0\n\t"
      ".set dp_more, 1\n\t"
      ".irpc ch, \"\\tuple\"\n\t"
      ".if '\\ch' == ':'\n\t.set dp_more, 0\n\t.endif\n\t"
      ".if dp_more && '\\ch' >= '0' && '\\ch' <= '9'\n\t"
      ".set dp_first, 10 * dp_first + ('\\ch' - '0')\n\t.endif\n\t"
      ".endr\n\t"
      ".irp i, 0, 1, 2, 3\n\t"
      "v_mul_f32 v[dp_first+\\i], %[f], v[dp_first+\\i]\n\t"
      ".endr\n\t"
      ".endr\n\ts_nop 1\n.Lkeep%=:"
      : "+v"(c[0][0]), "+v"(c[0][1]), "+v"(c[1][0]), "+v"(c[1][1])
      : [turn] "s"(turn), [f] "s"(f)
      : "scc");
}

// w: the weights of the first 64 samples, one a lane.  Returns the weight that the sums are expressed in (0: no sample counts).
template <bool F16>
__device__ __forceinline__ float tn_weighted_small(const GroupLayer& ly, int B, const float* C, float w, int m0, int n0,
                                                   unsigned lds0, f32x4 (&acc)[2][2]) {
  using S = SmallTile;
  const int d = ly.d_in, p = ly.d_out, blocks = (ly.T + S::BK - 1) / S::BK;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  // global -> LDS: a wave's load is rows 8 wave .. 8 wave + 7 of the k-block; chunks as for weighted_tiles, in rows of 128 bytes
  const int lrow = 8 * wave + (lane >> 3);
  const int chunk = (lane & 7) ^ ((lrow & 2) << 1 | (lrow >> 3 & 1) << 1);
  const unsigned a_org = m0 + chunk * 8 < d ? (unsigned)(lrow * d + m0 + chunk * 8) * 2u : OOB;
  const unsigned b_org = n0 + chunk * 8 < p ? (unsigned)(lrow * p + n0 + chunk * 8) * 2u : OOB;
  const unsigned a_slab = (unsigned)ly.T * d * 2u, b_slab = (unsigned)ly.T * p * 2u;
  const unsigned a_step = 2u * S::BK * d, b_step = 2u * S::BK * p;
  const unsigned lds_ld = lds0 + wave * 1024;
  uint64_t p_mask = 1;
  i32x4 ra, rb;
  unsigned va, vb;
  int p_left, p_stage;
  auto prefetch_a = [&]() { load_to_lds(ra, va, 0, lds_ld + p_stage * S::STAGE_BYTES); };
  auto prefetch_b = [&]() { load_to_lds(rb, vb, 0, lds_ld + p_stage * S::STAGE_BYTES + S::TILE_BYTES); };
  auto next_slab = [](i32x4& r, uint64_t bytes) {
    const uint64_t q = ((uint64_t)(uint32_t)r[1] << 32 | (uint32_t)r[0]) + bytes;
    r[0] = (int)(uint32_t)q;
    r[1] = (int)(uint32_t)(q >> 32);
  };
  auto prefetch_advance = [&]() {
    p_stage = p_stage + 1 == S::NSTAGE ? 0 : p_stage + 1;
    va += a_step;
    vb += b_step;
    if (--p_left == 0) {
      p_left = blocks;
      va = a_org;
      vb = b_org;
      p_mask >>= 1;
      if (p_mask == 0) {                                 // zeros from here on, the same number of loads
        ra[2] = rb[2] = 0;
        p_left = INT32_MAX;
      } else {
        const int n = __builtin_ctzll(p_mask);           // samples that do not count
        p_mask >>= n;
        next_slab(ra, (uint64_t)(n + 1) * a_slab);
        next_slab(rb, (uint64_t)(n + 1) * b_slab);
      }
    }
  };
  // LDS -> operands
  const int s = lane & 15;
  const int rrow = 8 * (lane >> 4) + (s >> 2);
  const int sw = (rrow & 2) << 1 | (rrow >> 3 & 1) << 1;
  const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
  const unsigned a_rd = lds0 + rrow * S::ROW_BYTES + ((((wm + 4 * (s & 3)) >> 3) ^ sw) << 4) + (s & 1) * 8;
  const unsigned b_rd = lds0 + S::TILE_BYTES + rrow * S::ROW_BYTES + ((((wn + 4 * (s & 3)) >> 3) ^ sw) << 4) + (s & 1) * 8;
  Frag fa[4][2], fb[4][2];                               // sets of two k-blocks in use and of the next two
  auto read_frag = [&](Frag& f, unsigned rd, int i, int stage) {
    unsigned base = stage * S::STAGE_BYTES;
    asm("" : "+s"(base));
    const unsigned addr = (rd ^ (unsigned)(i << 5)) + base;
    f.h[0] = lds_read_tr(addr);
    f.h[1] = lds_read_tr(addr + 4 * S::ROW_BYTES);
  };
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) acc[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr unsigned kOne = 0x3f800000u;
  int c_stage;
  unsigned f, turn;
  // Two k-blocks: wait for the next two, barrier.
  auto pair = [&](auto parity, auto next) {
    constexpr int P = decltype(parity)::value;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S::NSTAGE - 6) * 2) : "memory");
    __builtin_amdgcn_s_barrier();
    DP_PIN();
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      scale_if(turn, f, acc);
      DP_PIN();
      const int use = 2 * P + k, fill = 2 * (P ^ 1) + k;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int x = q & 1, y = q >> 1;
        acc[x][y] = mfma16<F16>(fb[use][y].v, fa[use][x].v, acc[x][y]);
        DP_PIN();
        if (q < 2)
          read_frag(fa[fill][q], a_rd, q, c_stage);
        else
          read_frag(fb[fill][q - 2], b_rd, q - 2, c_stage);
        if (q == 1) prefetch_a();
        if (q == 2) prefetch_b();
        if (q == 3) next();
        DP_PIN();
      }
      c_stage = c_stage + 1 == S::NSTAGE ? 0 : c_stage + 1;
    }
  };
  float held = 0.f;
#pragma unroll 1
  for (unsigned window = 0; window < (unsigned)B; window += 64) {
    if (window > 0) w = window_weights(C, window, B);
    const uint64_t mask = __ballot(w != 0.f && window + lane < (unsigned)B);
    if (mask == 0) continue;
    if (held != 0.f) __syncthreads();                    // the last window's fragments are read
    const int first = __builtin_ctzll(mask);
    p_mask = mask >> first;
    p_left = blocks;
    p_stage = c_stage = 0;
    va = a_org;
    vb = b_org;
    ra = make_rsrc(static_cast<const unsigned char*>(ly.a) + (size_t)(window + first) * a_slab, a_slab);
    rb = make_rsrc(static_cast<const unsigned char*>(ly.g) + (size_t)(window + first) * b_slab, b_slab);
#pragma unroll 1
    for (int q = 0; q < S::NSTAGE - 2; ++q) {
      prefetch_a();
      prefetch_b();
      prefetch_advance();
    }
    float ratio = 1.f;
    if (B > 1) {
      const uint64_t before = mask & ((1ull << lane) - 1);
      const float prev = __shfl(w, before ? 63 - __builtin_clzll(before) : lane);
      ratio = before ? prev / w : held != 0.f ? held / w : 1.f;
    }
    held = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w), 63 - __builtin_clzll(mask)));
    f = __builtin_amdgcn_readlane(__float_as_uint(ratio), first);
    turn = f ^ kOne;
    uint64_t rest = mask;                                // samples from the one at hand on
    int left = blocks;
    auto next = [&]() {
      prefetch_advance();
      turn = 0;
      if (--left == 0) {
        left = blocks;
        rest &= rest - 1;
        f = rest ? __builtin_amdgcn_readlane(__float_as_uint(ratio), __builtin_ctzll(rest)) : kOne;
        turn = f ^ kOne;
      }
    };
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S::NSTAGE - 4) * 2) : "memory");
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        read_frag(fa[k][q], a_rd, q, k);
        read_frag(fb[k][q], b_rd, q, k);
      }
    c_stage = 2;                                         // of the reads
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    // An odd number of blocks: one more of zeros, past the stream's end.
#pragma unroll 1
    for (int n = __builtin_popcountll(mask) * blocks; n > 0; n -= 4) {
      pair(even, next);
      if (n > 2) pair(odd, next);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // zero-fill loads past the end
  }
  return held;
}

}  // namespace dpbk
