// Internal declarations shared by the library's translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "dp_bk.h"
#include "philox.h"

namespace dpbk {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define DP_LDS(T, p) ((__attribute__((address_space(3))) T*)(p))

// One 32x32x16 matrix-core step on 16-bit operands with fp32 accumulation.  The kernels move
// operands as opaque 16-bit values (typed bf16x8 for convenience); F16 says the bits are IEEE
// binary16 rather than bfloat16, which only changes the instruction that multiplies them.
template <bool F16>
__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b),
                                                  c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// One 16x16x32 step: the same additions in the same order as two 32x32x16 steps, at less power.
template <bool F16>
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  if constexpr (F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Up to this many layers travel in one launch's kernel arguments.  (Larger groups work - the
// runtime takes 16 KiB of kernel arguments - but a single launch of cfg2's 144 layers measured
// 1 % slower in the gradient than three launches of 48, and no faster in the norms.)
constexpr int kMaxGroup = 48;

// One layer of a grouped launch.  tile_begin is the first workgroup of the layer.
struct GroupLayer {
  const void* a;
  const void* g;
  float* out;       // gradient [d_in, d_out] (clipped_grad) or unused
  int T, d_in, d_out;
  int path;
  int tile_begin;   // first block index that belongs to this layer
  int sq_index;     // layer number within the caller's stack (row of sqnorm)
  int part_begin;   // first partial-sum slot of this layer in the workspace
  int tiles_per_sample;
  int c_off;        // gradient kernels: this layer's weights are C[c_off + i] (its clipping group)
  int stream;       // matrix-core gradient kernels: rows leave by streaming stores (not of an accumulating launch)
};

struct GroupArgs {
  int n_layers;
  int total_blocks;
  int B;
  int accumulate;
  int f16;          // operands are IEEE binary16 (else bfloat16)
  GroupLayer layer[kMaxGroup];
};

// Noise added in the epilogue of the large-tile gradient kernels (eq. (1) of the paper):
// element j of layer l's gradient has global index layer_off[l] + j and receives
// stddev * z_index when lo <= index < hi.  stddev == 0 switches the noise off.
struct NoiseArgs {
  float stddev;
  uint32_t step_lo, step_hi;
  uint64_t lo, hi;
  RoundKeys rk;
  uint64_t layer_off[kMaxGroup];
};

// What the kernels that finish squared norms make of them.
//  kLayerFactors: one group per layer: the factor of each norm as it is written (R[j]: threshold of the launch's layer j;
//    C_out as large as the whole stack's norms).
//  kGroupFactors: one group of all L rows of the call: the workgroup that ends last (of `blocks`, counted in
//    *counter, which is zero before and after) adds the rows up and writes C_out[B] and norm_out[B] (or nullptr).
constexpr int kFinishLanes = 4096;     // kGroupFactors: B * width at most
enum ClipKind { kNoFactors = 0, kLayerFactors = 1, kGroupFactors = 2 };
struct NormClip {
  int kind;
  int mode;
  float stability;
  float* C_out;
  float* norm_out;
  unsigned* counter;
  unsigned blocks;
  int L, width;                 // width: lanes to a sample, a power of two, 64 or no less than L
  float R[kMaxGroup];           // kGroupFactors: R[0]
};

// The layer that owns workgroup (or tile) number `id`: the last one whose tile_begin is <= id.  Called by whole waves: a
// lane looks at each layer, one load's latency.  (A search by halves is a chain of six: 3 x 18 tokens, 48 layers of width 320
// 33.5 us a step with it, 30.6 without; 24 adapter pairs of 768 x 16 86.0 and 83.7.)
__device__ __forceinline__ int layer_of(const GroupArgs& ga, int id) {
  static_assert(kMaxGroup <= 64, "a lane to a layer");
  const int lane = threadIdx.x & 63;
  const int begin = ga.layer[lane < ga.n_layers ? lane : 0].tile_begin;
  return __builtin_popcountll(__ballot(lane < ga.n_layers && begin <= id)) - 1;
}

// The fp32 norm kernel runs one workgroup per (layer, sample); layers whose norm needs more
// multiply-adds per sample than this are refused (DP_ERR_UNSUPPORTED) instead of holding one
// compute unit for long.
constexpr int64_t kF32MaxWork = (int64_t)1 << 28;

inline dp_status hip_status(hipError_t e) { return e == hipSuccess ? DP_OK : DP_ERR_HIP; }

// A launch takes less than 2^32 work items in a dimension (beyond it workgroups go missing without an error).
// Kernels whose workgroups of 512 threads can come in larger numbers (2^23: one per sample of a stack, or per
// tile of a layer of 1 x 2^28) are launched in runs: workgroup first + blockIdx.x of n.  (A second grid
// dimension needs a test for the numbers past n, which put 0.6 us on a gradient kernel of 12 us.)
template <class F>
dp_status launch_in_runs(int64_t n, F launch) {
  constexpr int64_t kRun = (int64_t)1 << 22;
  for (int64_t first = 0; first < n; first += kRun) {
    launch(dim3((unsigned)(n - first < kRun ? n - first : kRun)), (int)first);
    const dp_status st = hip_status(hipGetLastError());
    if (st != DP_OK) return st;
  }
  return DP_OK;
}

// Kernels that need more than 64 KiB of LDS must be told so once per device; `done` is the
// caller's per-kernel table of devices already prepared.  These tables are the library's only
// mutable host state: flags that go from false to true once, so two threads that race on one at
// worst both make the (idempotent) attribute call.
constexpr int kMaxDevices = 64;
using ReadyTable = std::atomic<bool>[kMaxDevices];
template <class K>
dp_status allow_big_lds(K kernel, int bytes, ReadyTable& done) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return DP_ERR_HIP;
  if (done[dev].load(std::memory_order_acquire)) return DP_OK;
  dp_status st = hip_status(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                                hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
  if (st == DP_OK) done[dev].store(true, std::memory_order_release);
  return st;
}

// --- launchers implemented in the .hip files (all validate nothing; callers did) ---
dp_status launch_noise(float* grad, uint64_t global_offset, uint64_t count, float stddev,
                       uint64_t seed, uint64_t step, hipStream_t s);
dp_status launch_philox_blocks(uint32_t* out, uint64_t first_block, uint64_t n_blocks,
                               uint64_t seed, uint64_t step, hipStream_t s);
dp_status launch_clip_factors(const float* sqnorm, int L, int B, int mode, float R, float stability,
                              float* C_out, float* norm_out, hipStream_t s);
// norm_reduce of the launch's layers (launch_norm_reduce_group) and the clip factors of all L rows in one launch, the same
// bits; norm_clip_supports: L is not beyond its LDS.
bool norm_clip_supports(int L);
dp_status launch_norm_clip(const GroupArgs& ga, const float* partials, float* sqnorm, int L, int mode, float R,
                           float stability, float* C_out, float* norm_out, hipStream_t s);
dp_status launch_clip_factors_grouped(const float* sqnorm, int B, const int32_t* group_begin, int M,
                                      const float* R, int mode, float stability, float* C_out,
                                      float* norm_out, hipStream_t s);
dp_status launch_bias_norm(const void* g, dp_dtype dt, int B, int T, int p, float* colsum,
                           float* sqnorm_out, hipStream_t s);
dp_status launch_clipped_bias_grad(const float* colsum, int B, int p, const float* C, float* grad_b,
                                   int accumulate, hipStream_t s);

// fp32 kernels (fp32_kernels.hip), grouped over layers.  Norms: ga.layer[j].path selects the form, one
// workgroup per (layer, sample).  Gradients: tile_begin = first workgroup (clipped_grad_f32_tiles per layer),
// c_off; na.stddev == 0: no noise.
int64_t clipped_grad_f32_tiles(int d, int p);
dp_status launch_norms_f32_group(const GroupArgs& ga, float* sqnorm, const NormClip& nc, hipStream_t s);
dp_status launch_clipped_grad_f32_group(const GroupArgs& ga, const float* C, const NoiseArgs& na, hipStream_t s);

// Tiles of tn_pipeline.h.  A launch runs in rounds of the tiles that are resident at a time: 256 large ones
// (one per compute unit) or 512 of 128 x 128 (two), and a round of the latter, half the work, takes three
// fifths of the time (measured on 1024-wide layers, 2048 tokens: 57 us and 34 us).  So large tiles
// where they come in whole rounds, small ones where few tiles or padding would leave large ones idle.
// The instantiated norms price rounds so at every width; of the gradients' launches only those over rows of whole 128-byte lines
// or few rows (clipped_grad_tail: 0.65 to 1.0 of a large round elsewhere).
constexpr int kBigRound = 256, kMidRound = 512;
constexpr int kBigRoundCost = 5, kMidRoundCost = 3;

// bf16 MFMA kernels, grouped over layers.
int ghost_tiles_per_sample(int T);
int perex_tiles_per_sample(int d, int p);
int clipped_grad_tiles(int d, int p);
dp_status launch_ghost_group(const GroupArgs& ga, float* partials, hipStream_t s);
dp_status launch_perex_group(const GroupArgs& ga, float* partials, hipStream_t s);
// With direct global->LDS loads, three k-blocks ahead (perex_dma.hip); tiles of 128 x 128 as above or, `big`,
// of 256 x 256 (ga laid out for clipped_grad_big_tiles tiles per sample, partial sums as above: the same bits).
bool perex_dma_supports(int T, int d, int p);
dp_status launch_perex_dma_group(const GroupArgs& ga, float* partials, bool big, hipStream_t s);
// Narrow layers on tiles of the 128 x 128 ones' numbering (perex_narrow.hip).
bool perex_narrow_supports(int T, int d, int p);
dp_status launch_perex_narrow_group(const GroupArgs& ga, float* partials, hipStream_t s);
dp_status launch_norm_reduce_group(const GroupArgs& ga, const float* partials, float* sqnorm_out,
                                   const NormClip& nc, hipStream_t s);
dp_status launch_clipped_grad_group(const GroupArgs& ga, const float* C, hipStream_t s);
// 256x128-tile ghost-norm kernel with direct global->LDS loads (ghost_big.hip).
int ghost_big_tiles_per_sample(int T);
bool ghost_big_supports(int T, int d, int p);
dp_status launch_ghost_big_group(const GroupArgs& ga, float* partials, hipStream_t s);
// Whole-sample ghost-norm kernel for 129 .. 256 tokens (ghost_sample.hip): one workgroup per sample, final
// squared norms.
bool ghost_sample_supports(int T, int d, int p);
dp_status launch_ghost_sample_group(const GroupArgs& ga, float* sqnorm, const NormClip& nc, hipStream_t s);
// Samples of up to 32 tokens, several to a workgroup, final squared norms (ghost_brief.hip):
// ga.layer[j].tiles_per_sample = workgroups to 32 rows, up to ghost_brief_max_parts, tile_begin = first workgroup.
bool ghost_brief_supports(int T);
int64_t ghost_brief_blocks(int B, int T, int parts);
int ghost_brief_max_parts(int B, int T);
dp_status launch_ghost_brief_group(const GroupArgs& ga, float* sqnorm, const NormClip& nc, hipStream_t s);
// 33 to 64 tokens of not too wide layers, a workgroup to a sample (ghost_brief.hip): final norms too.
bool ghost_pair_supports(int T, int d, int p);
dp_status launch_ghost_pair_group(const GroupArgs& ga, float* sqnorm, const NormClip& nc, hipStream_t s);
// 256x256-tile kernel with direct global->LDS loads (grad_gemm.hip).
int clipped_grad_big_tiles(int d, int p);
int64_t clipped_grad_mid_tiles(int d, int p);
// Of a launch of n large tiles whose layers hold n_mid tiles of 128 x 128 and contract over up to `rows` rows, how many
// (the last ones) are cut into side x side sub-tiles (whole_lines: every row of every operand is whole 128-byte lines; long_off_sectors: rows of
// some operand begin off 64-byte pieces of memory, and no sample is short); brief: on the 128 x 128 tiles of short contractions.
constexpr int kGradMidSide = 2, kGradTailSide = 4;
struct GradTail {
  int tiles, side;
  bool brief;
};
GradTail clipped_grad_tail(int n, int64_t n_mid, int64_t rows, bool whole_lines, bool long_off_sectors, bool out16);
// The launches of a group on these tiles.  blocks: in whole k-blocks (tn_weighted.h); workgroups: of the tiles that are not cut,
// each one or more of them.
struct GradLaunches {
  GradTail cut;
  bool blocks;
  int workgroups;
};
GradLaunches clipped_grad_launches(const GroupArgs& ga, bool out16);
bool clipped_grad_big_supports(int T, int d, int p);
// noise == nullptr: gradients only.  out16: the layers' `out` pointers address 16-bit arrays of the
// operands' storage type (bf16 or fp16) instead of fp32.
dp_status launch_clipped_grad_big_group(const GroupArgs& ga, const float* C, const NoiseArgs* noise,
                                        hipStream_t s, bool out16 = false);

// Contraction over the packed rows of all samples (grad_packed.hip): ga.layer[j].path =
// grad_packed_shape(d, p), tile_begin = first workgroup (grad_packed_tiles per layer).
int grad_packed_shape(int d, int p);
int grad_packed_tiles(int d, int p);
bool grad_packed_supports(int B, int T, int d, int p);
dp_status launch_grad_packed_group(const GroupArgs& ga, const float* C, const NoiseArgs* noise, hipStream_t s);

// Clip-weighted sum of kept per-sample gradients (kept.hip).  ga.layer[j]: a = kept [B, d * p] fp32,
// out = grad, tile_begin = first workgroup (kept_blocks(d, p) per layer), c_off; noise as NoiseArgs,
// layer_off[j] == ~0 switching it off for layer j.
int kept_blocks(int d, int p);
dp_status launch_kept_weighted_sum(const GroupArgs& ga, const float* C, const NoiseArgs& na, hipStream_t s);

// Layer-wise clipping in one pass for layers that fit one workgroup tile (layerwise.hip).
// Shape class of a d x p layer (0: up to 128 x 128, 1: up to 512 x 32, 2: up to 32 x 512), or -1.
int layerwise_fused_shape(int d, int p);
// ga.layer[j]: tile_begin = first workgroup, tiles_per_sample = sample chunks, part_begin = float
// offset of the layer's [chunks][d * p] sums in `partial`, sq_index = row of sqnorm / C_out.
dp_status launch_layerwise_fused(int shape, const GroupArgs& ga, const float* R, int mode, float stability, float* partial,
                                 float* sqnorm, float* C_out, hipStream_t s);
// ga.layer[j].out (+)= the layer's chunks added in order (+ noise when na.stddev != 0).
dp_status launch_layerwise_reduce(const GroupArgs& ga, const float* partial, const NoiseArgs& na, hipStream_t s);

}  // namespace dpbk
