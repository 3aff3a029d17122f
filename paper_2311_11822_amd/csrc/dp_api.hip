// Host side of the C ABI: argument validation, grouping of layers into launches.
// No device code lives here and no device memory is allocated.
#include <math.h>
#include <algorithm>
#include <vector>

#include "dp_internal.h"
#include "tile_order.h"

using namespace dpbk;

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool dtype_ok(dp_dtype dt) { return dt == DP_F32 || dt == DP_BF16 || dt == DP_F16; }

bool dims_ok(dp_dtype dt, int B, int T, int d, int p) {
  if (B <= 0 || T <= 0 || d <= 0 || p <= 0) return false;
  if (dt != DP_F32 && ((d & 7) || (p & 7))) return false;      // 16-bit rows must be 16-byte multiples
  // index arithmetic inside the kernels is 64-bit for element offsets, 32-bit per dimension
  if ((int64_t)B * T > INT32_MAX) return false;
  return true;
}

dp_status check_layer_ptrs(const void* a, const void* g) {
  if (!a || !g) return DP_ERR_INVALID_ARG;
  if (!aligned16(a) || !aligned16(g)) return DP_ERR_INVALID_ARG;
  return DP_OK;
}

// Ghost layers of more than 64 tokens (wide ones: 32) that the large-tile kernel can address; up to 128 tokens the 128 x 128-tile kernel
// takes them too (ghost_stays_small), with the same bits.
bool ghost_uses_big(const dp_layer& ly) {
  return !ghost_brief_supports(ly.T) && !ghost_pair_supports(ly.T, ly.d_in, ly.d_out) && ghost_big_supports(ly.T, ly.d_in, ly.d_out);
}

// Up to 128 tokens a sample is one workgroup in either kernel.  The large-tile kernel keeps deeper prefetch and has a
// compute unit to itself; of the other two share one, and a round of these 512 takes 5/3 of the time of 256 large
// ones (112 tokens, d_in + d_out = 912: 25.1 and 15.3 us).  So the rounds decide, but narrow layers, whose samples are
// over before a deep prefetch pays, stay on the small kernel beyond one round (d_in + d_out = 272: 12.5 and 9.7 us a
// round), and wide ones on the large kernel (2096: 43.5 and 24.4).  512 samples 24 + 16 wide: 10.0 us here, 13.3 on the
// large kernel, 2048 of 392 + 296: 80 and 94; 768 of 760 + 520: 49.5 and 45.9.
// From 96 tokens on, whole 64-wide k-blocks: the large kernel, which has no edge handling there.
// Below 96 tokens either kernel pays for 128, so the same rounds; which of them is decided for the call by its widest layer,
// one launch instead of two.  Norms of 80 tokens, us, small and large kernel: 7 samples of five layers 512 + 512 18.7, 12.3;
// 4 of 1024 + 3072 .. 4096 67.0, 31.8; 10 of 24 layers 1472 + 4416 .. 5888 94.8, 49.1; 32 of twelve 768 + 2304 .. 3072 61.2, 49.1;
// of 90 tokens: 96 of eight 760 + 520 46.5, 40.1; 320 samples of 392 + 296 17.8, 20.3; 2048 of 128 + 384 .. 512 45.8, 55.9.
bool ghost_stays_small(const dp_layer& ly, int64_t samples, int64_t widest) {
  if (ly.T > 128 || (ly.T >= 96 && ly.d_in % 64 == 0 && ly.d_out % 64 == 0)) return false;
  const int64_t width = ly.T >= 96 ? (int64_t)ly.d_in + ly.d_out : widest;
  if (samples <= 256 || width >= 1800) return false;
  return width < 500 || 3 * ((samples + 255) / 256) >= 5 * ((samples + 511) / 512);
}

// Samples of 129 .. 256 tokens take the kernel that holds a whole sample in one workgroup.
bool ghost_uses_sample(const dp_layer& ly) { return ghost_sample_supports(ly.T, ly.d_in, ly.d_out); }

int tiles_per_sample(int path, const dp_layer& ly) {
  if (path == DP_PATH_PEREX) return perex_tiles_per_sample(ly.d_in, ly.d_out);
  if (ghost_uses_sample(ly)) return 1;
  return ghost_uses_big(ly) ? ghost_big_tiles_per_sample(ly.T) : ghost_tiles_per_sample(ly.T);
}

// Instantiated norm on n_big tiles of 256 x 256 or n_mid of 128 x 128?
bool perex_on_big_tiles(int64_t n_big, int64_t n_mid) {
  return kBigRoundCost * ((n_big + kBigRound - 1) / kBigRound) < kMidRoundCost * ((n_mid + kMidRound - 1) / kMidRound);
}

// Clip factors that the norm launches form on the way.
struct ClipSpec {
  int mode;
  float stability;
  float* C_out;
  const float* layer_R;          // layer-wise: thresholds by layer of the call; nullptr: all layers in one group
  float R;                       // one group
  float* norm_out;
  unsigned* counter;             // one group: device, zero between the calls; or nullptr
};

// One group: the last launch of partial sums, not added up yet.
struct PendingReduce {
  GroupArgs ga;
  bool any = false;
};

// For the kernels' arguments, layer-wise thresholds still to be filled in.
NormClip layer_clip(const ClipSpec* clip) {
  NormClip nc = {};
  nc.kind = clip && clip->layer_R ? kLayerFactors : kNoFactors;
  if (!clip) return nc;
  nc.mode = clip->mode;
  nc.stability = clip->stability;
  nc.C_out = clip->C_out;
  return nc;
}

// The last launch of final norms forms the factors of the one group where that is cheaper than a launch.  A launch costs the
// host 3 us of a step; the count, workgroups after each other in one cell, costs the GPU from 0.1 us at 100 to 1.9 at 250
// workgroups more than the launch.  So: few workgroups and layers, or a step so small that the host bounds it (it takes
// 20 us from Python).  A step, us, factors here and in a launch.  Below the line: seven fp32 layers 16 x 16 of 14 x 39 tokens
// 18.6 and 23.1, twelve bf16 64 x 64 of 10 x 32 20.7 and 23.6, 24 fp16 384 x 32 of 7 x 32 (5.7 MB) 20.9 and 23.7, 22 bf16
// 64 x 32 of 8 x 24 20.2 and 23.5; at its worst eight fp32 58 x 58 of 17 x 35 31.8 and 31.5.  Above it: eleven bf16
// 256 x 256 of 17 x 17 (6.1 MB) 27.3 and 25.9, 22 fp16 696 x 48 of 11 x 32 28.2 and 26.5, four bf16 128 x 40 of 56 x 31
// (2.4 MB, but a chain of 1736 rows) 45.8 and 44.1, nine fp16 112 x 112 of 16 x 23 (twice the matrix instructions a row)
// 25.2 and 24.5.  fp32 layers take longer for a byte: four 76 to 304 wide of 25 x 18 (2.5 MB) 21.9 and 23.3.
constexpr int kLastCost = 96, kLastBlocks = 256, kLastLayers = 256;
int lanes_for(int L) {
  int width = 1;
  while (width < 64 && width < L) width *= 2;
  return width;
}

bool host_bounds_step(const dp_layer* layers, int L, dp_dtype dt, int B) {
  const int64_t size = dt == DP_F32 ? 4 : 2, most_bytes = dt == DP_F32 ? 3000000 : 6000000;
  const int64_t most_rows = dt == DP_F32 ? 1024 : dt == DP_BF16 ? 512 : 256;
  int64_t bytes = 0;
  for (int l = 0; l < L && bytes <= most_bytes; ++l) {
    const int64_t rows = (int64_t)B * layers[l].T, d = layers[l].d_in, p = layers[l].d_out;
    if (rows > most_rows || d > most_bytes || p > most_bytes) return false;      // the sums below stay far from 2^63
    bytes += rows * (d + p) * size + 4 * d * p;
  }
  return bytes <= most_bytes;
}

bool last_forms_factors(const ClipSpec* clip, int64_t blocks, const dp_layer* layers, int L, dp_dtype dt, int B) {
  return clip && !clip->layer_R && clip->counter && blocks <= kLastBlocks && L <= kLastLayers &&
         (int64_t)B * lanes_for(L) <= kFinishLanes && (blocks + L <= kLastCost || host_bounds_step(layers, L, dt, B));
}

void set_group_factors(NormClip& nc, const ClipSpec& clip, int64_t blocks, int L) {
  nc.kind = kGroupFactors;
  nc.norm_out = clip.norm_out;
  nc.counter = clip.counter;
  nc.blocks = (unsigned)blocks;
  nc.L = L;
  nc.width = lanes_for(L);
  nc.R[0] = clip.R;
}

// Workgroups to 32 rows in the brief kernel: one, or two, four ... while all of them have a compute unit of their own.
// (Two of a compute unit measured the same: 256 and 512 workgroups of one-token samples 107.8 and 107.6 us a step.)
// Returns the workgroups of the launch.
constexpr int kBriefBlocks = 256;
int64_t share_brief_samples(GroupArgs& ga) {
  int64_t blocks = 0;
  for (int parts = 1;; parts *= 2) {
    int64_t n = 0;
    bool more = false;
    for (int j = 0; j < ga.n_layers; ++j) {
      const int most = ghost_brief_max_parts(ga.B, ga.layer[j].T);
      more = more || parts < most;
      n += ghost_brief_blocks(ga.B, ga.layer[j].T, std::min(parts, most));
    }
    if (parts > 1 && n > kBriefBlocks) return blocks;
    blocks = n;
    n = 0;
    for (int j = 0; j < ga.n_layers; ++j) {
      GroupLayer& gl = ga.layer[j];
      gl.tiles_per_sample = std::min(parts, ghost_brief_max_parts(ga.B, gl.T));
      gl.tile_begin = (int)n;
      n += ghost_brief_blocks(ga.B, gl.T, gl.tiles_per_sample);
    }
    if (!more) return blocks;
  }
}

// Launches the norm kernels of one path for the listed layers, in chunks of kMaxGroup.
// part_begin[l] is the layer's first slot in the partial-sum workspace.  last_rows: rows of the whole call if these are
// its last norm launches (0: not); *formed: the last of them formed the factors.
enum NormKernel { kGhostBig = 0, kGhostSmall = 1, kPerex = 2, kGhostSample = 3, kGhostBrief = 4, kPerexNarrow = 5, kGhostPair = 6 };
constexpr int kNormKernels = 7;

dp_status run_norm_path(NormKernel kernel, const dp_layer* layers, int* which, int n_which,
                        const int64_t* part_begin, dp_dtype dt, int B, float* partials,
                        float* sqnorm_out, hipStream_t s, const int* row_of, float* const* kept,
                        const ClipSpec* clip, PendingReduce* pending, int last_rows, bool* formed) {
  // A tile's length is the contraction it runs over (d_in + d_out for the ghost norm, T for the
  // instantiated one).  Longest first: workgroups are handed out in order, so the short tiles
  // fill the end of the launch.  Each layer writes its own workspace slots and sqnorm row, so
  // the order inside a launch is free.  (Stable insertion sort in place: this path must not
  // touch the heap, see dp_norms_multi_static.)
  auto length = [&](int l) {
    return kernel == kPerex || kernel == kPerexNarrow ? (int64_t)layers[l].T : (int64_t)layers[l].d_in + layers[l].d_out;
  };
  for (int i = 1; i < n_which; ++i) {
    const int x = which[i];
    int j = i;
    for (; j > 0 && length(which[j - 1]) < length(x); --j) which[j] = which[j - 1];
    which[j] = x;
  }
  for (int begin = 0; begin < n_which; begin += kMaxGroup) {
    GroupArgs ga;
    NormClip nc = layer_clip(clip);
    ga.B = B;
    ga.accumulate = 0;
    ga.f16 = dt == DP_F16;
    ga.n_layers = std::min(kMaxGroup, n_which - begin);
    int64_t blocks = 0;
    for (int j = 0; j < ga.n_layers; ++j) {
      const int l = which[begin + j];
      GroupLayer& gl = ga.layer[j];
      if (nc.kind == kLayerFactors) nc.R[j] = clip->layer_R[l];
      gl.a = layers[l].a;
      gl.g = layers[l].g;
      gl.out = (kernel == kPerex || kernel == kPerexNarrow) && kept ? kept[l] : nullptr;
      gl.T = layers[l].T;
      gl.d_in = layers[l].d_in;
      gl.d_out = layers[l].d_out;
      gl.path = layers[l].path;
      gl.tile_begin = (int)blocks;
      gl.sq_index = row_of ? row_of[l] : l;
      gl.part_begin = (int)part_begin[l];
      gl.tiles_per_sample = tiles_per_sample(gl.path, layers[l]);
      gl.c_off = 0;
      blocks += (int64_t)gl.tiles_per_sample * B;
    }
    if (kernel == kGhostBrief) blocks = share_brief_samples(ga);
    ga.total_blocks = (int)blocks;
    if (kernel == kGhostBrief || kernel == kGhostSample || kernel == kGhostPair) {       // final norms: nothing to add up
      if (last_rows && begin + kMaxGroup >= n_which && last_forms_factors(clip, blocks, layers, last_rows, dt, B)) {
        set_group_factors(nc, *clip, blocks, last_rows);
        *formed = true;
      }
      dp_status st = kernel == kGhostBrief  ? launch_ghost_brief_group(ga, sqnorm_out, nc, s)
                     : kernel == kGhostPair ? launch_ghost_pair_group(ga, sqnorm_out, nc, s)
                                            : launch_ghost_sample_group(ga, sqnorm_out, nc, s);
      if (st != DP_OK) return st;
      continue;
    }
    // instantiated norm: the kernel with the deep load pipeline unless a slab is beyond its
    // 32-bit addressing, on large tiles (with the same partial sums) where they pay
    bool dma = kernel == kPerex, big = false;
    for (int j = 0; j < ga.n_layers; ++j)
      dma = dma && perex_dma_supports(ga.layer[j].T, ga.layer[j].d_in, ga.layer[j].d_out);
    if (dma) {
      int64_t n = 0;
      for (int j = 0; j < ga.n_layers; ++j) n += (int64_t)clipped_grad_big_tiles(ga.layer[j].d_in, ga.layer[j].d_out) * B;
      big = perex_on_big_tiles(n, blocks);
      if (big) {
        blocks = 0;
        for (int j = 0; j < ga.n_layers; ++j) {
          GroupLayer& gl = ga.layer[j];
          gl.tile_begin = (int)blocks;
          gl.tiles_per_sample = clipped_grad_big_tiles(gl.d_in, gl.d_out);
          blocks += (int64_t)gl.tiles_per_sample * B;
        }
        ga.total_blocks = (int)blocks;
      }
    }
    dp_status st = kernel == kGhostBig      ? launch_ghost_big_group(ga, partials, s)
                   : kernel == kGhostSmall  ? launch_ghost_group(ga, partials, s)
                   : kernel == kPerexNarrow ? launch_perex_narrow_group(ga, partials, s)
                   : dma                    ? launch_perex_dma_group(ga, partials, big, s)
                                            : launch_perex_group(ga, partials, s);
    if (st != DP_OK) return st;
    if (big)
      for (int j = 0; j < ga.n_layers; ++j)
        ga.layer[j].tiles_per_sample = perex_tiles_per_sample(ga.layer[j].d_in, ga.layer[j].d_out);
    if (pending) std::swap(pending->ga, ga);             // the launch before it, if any, is added up now
    if (!pending || pending->any) st = launch_norm_reduce_group(ga, partials, sqnorm_out, nc, s);
    if (st != DP_OK) return st;
    if (pending) pending->any = true;
  }
  return DP_OK;
}

// Total partial-sum slots, or -1 if a layer is invalid.
int64_t norm_slots(const dp_layer* layers, int L, dp_dtype dt, int B, int64_t* begin) {
  if (!layers || L <= 0 || B <= 0) return -1;
  int64_t total = 0;
  for (int l = 0; l < L; ++l) {
    if (!dims_ok(dt, B, layers[l].T, layers[l].d_in, layers[l].d_out)) return -1;
    if (layers[l].path != DP_PATH_GHOST && layers[l].path != DP_PATH_PEREX) return -1;
    if (begin) begin[l] = total;
    if (dt != DP_F32) total += (int64_t)tiles_per_sample(layers[l].path, layers[l]) * B;
    if (total > INT32_MAX) return -1;
  }
  return total;
}

// The factors of one group over all layers, together with the partial sums that wait, if there are any.
constexpr int kNormClipSamples = 1 << 20;                // workgroups of 1024 threads: one grid dimension
dp_status group_clip(const ClipSpec* clip, const PendingReduce* pending, float* sqnorm, const float* partials, int L, int B,
                     hipStream_t s) {
  if (!clip || clip->layer_R) return DP_OK;
  if (pending && pending->any)
    return launch_norm_clip(pending->ga, partials, sqnorm, L, clip->mode, clip->R, clip->stability, clip->C_out,
                            clip->norm_out, s);
  return launch_clip_factors(sqnorm, L, B, clip->mode, clip->R, clip->stability, clip->C_out, clip->norm_out, s);
}

// begin: room for L values; idx: room for kNormKernels * L values (the layers of each kernel).  The caller
// provides both so that this function never touches the heap.  row_of (or nullptr): layer l's
// squared norms go to row row_of[l] of sqnorm_out instead of row l.  clip (or nullptr): clip factors too, of each layer,
// or (row_of is nullptr then) of all together.
dp_status norms_impl(const dp_layer* layers, int L, dp_dtype dt, int B, float* sqnorm_out, void* ws,
                     size_t ws_bytes, hipStream_t s, int64_t* begin, int* idx, const int* row_of = nullptr,
                     float* const* kept = nullptr, const ClipSpec* clip = nullptr) {
  if (!dtype_ok(dt)) return DP_ERR_INVALID_ARG;
  if (!sqnorm_out) return DP_ERR_INVALID_ARG;
  const int64_t slots = norm_slots(layers, L, dt, B, begin);
  if (slots < 0) return DP_ERR_INVALID_ARG;
  for (int l = 0; l < L; ++l) {
    dp_status st = check_layer_ptrs(layers[l].a, layers[l].g);
    if (st != DP_OK) return st;
  }
  if (dt == DP_F32) {
    for (int l = 0; l < L; ++l) {
      const dp_layer& ly = layers[l];
      const __int128 work = ly.path == DP_PATH_GHOST
                                ? (__int128)ly.T * ly.T / 2 * ((int64_t)ly.d_in + ly.d_out)
                                : (__int128)ly.T * ly.d_in * ly.d_out;
      if (work > kF32MaxWork) return DP_ERR_UNSUPPORTED;
    }
    const int per_launch = std::max(1, std::min(kMaxGroup, INT32_MAX / 2 / B));
    bool formed = false;
    for (int l0 = 0; l0 < L; l0 += per_launch) {
      GroupArgs ga;
      NormClip nc = layer_clip(clip);
      ga.B = B;
      ga.accumulate = 0;
      ga.f16 = 0;
      ga.n_layers = std::min(per_launch, L - l0);
      for (int j = 0; j < ga.n_layers; ++j) {
        const dp_layer& ly = layers[l0 + j];
        GroupLayer& gl = ga.layer[j];
        gl = {};
        gl.a = ly.a;
        gl.g = ly.g;
        gl.T = ly.T;
        gl.d_in = ly.d_in;
        gl.d_out = ly.d_out;
        gl.path = ly.path;
        gl.sq_index = row_of ? row_of[l0 + j] : l0 + j;
        if (nc.kind == kLayerFactors) nc.R[j] = clip->layer_R[l0 + j];
      }
      ga.total_blocks = ga.n_layers * B;
      if (l0 + per_launch >= L && last_forms_factors(clip, ga.total_blocks, layers, L, dt, B)) {
        set_group_factors(nc, *clip, ga.total_blocks, L);
        formed = true;
      }
      dp_status st = launch_norms_f32_group(ga, sqnorm_out, nc, s);
      if (st != DP_OK) return st;
    }
    return formed ? DP_OK : group_clip(clip, nullptr, sqnorm_out, nullptr, L, B, s);
  }
  if (!ws || ws_bytes < (size_t)slots * sizeof(float)) return DP_ERR_WORKSPACE;
  if (!aligned16(ws)) return DP_ERR_INVALID_ARG;
  int* list[kNormKernels];
  for (int k = 0; k < kNormKernels; ++k) list[k] = idx + (size_t)k * L;
  int count[kNormKernels] = {};
  int64_t samples = 0, widest = 0;                       // that either large-tile or 128 x 128 kernel may take
  for (int l = 0; l < L; ++l)
    if (layers[l].path == DP_PATH_GHOST && ghost_uses_big(layers[l]) && layers[l].T <= 128) {
      samples += B;
      widest = std::max(widest, (int64_t)layers[l].d_in + layers[l].d_out);
    }
  for (int l = 0; l < L; ++l) {
    const bool narrow = perex_narrow_supports(layers[l].T, layers[l].d_in, layers[l].d_out);
    const int k = layers[l].path == DP_PATH_PEREX ? (narrow ? kPerexNarrow : kPerex)
                  : ghost_brief_supports(layers[l].T) ? kGhostBrief
                  : ghost_pair_supports(layers[l].T, layers[l].d_in, layers[l].d_out) ? kGhostPair
                  : ghost_uses_sample(layers[l])  ? kGhostSample
                  : ghost_uses_big(layers[l]) && !ghost_stays_small(layers[l], samples, widest) ? kGhostBig
                                                                                        : kGhostSmall;
    list[k][count[k]++] = l;
  }
  float* partials = static_cast<float*>(ws);
  PendingReduce held;
  PendingReduce* pending = clip && !clip->layer_R && B <= kNormClipSamples && norm_clip_supports(L) ? &held : nullptr;
  int last = kNormKernels - 1;
  while (count[last] == 0) --last;
  bool formed = false;
  for (int k = 0; k <= last; ++k) {
    const bool ends = k == last && !(pending && pending->any);
    dp_status st = run_norm_path((NormKernel)k, layers, list[k], count[k], begin, dt, B, partials, sqnorm_out, s,
                                 row_of, kept, clip, pending, ends ? L : 0, &formed);
    if (st != DP_OK) return st;
  }
  return formed ? DP_OK : group_clip(clip, pending, sqnorm_out, partials, L, B, s);
}

dp_status norms_impl(const dp_layer* layers, int L, dp_dtype dt, int B, float* sqnorm_out, void* ws,
                     size_t ws_bytes, hipStream_t s, const int* row_of = nullptr, float* const* kept = nullptr,
                     const ClipSpec* clip = nullptr) {
  if (!layers || L <= 0) return DP_ERR_INVALID_ARG;
  std::vector<int64_t> begin(L);
  std::vector<int> idx(kNormKernels * (size_t)L);
  return norms_impl(layers, L, dt, B, sqnorm_out, ws, ws_bytes, s, begin.data(), idx.data(), row_of, kept, clip);
}

dp_status single_norm(dp_path path, const void* a, const void* g, dp_dtype dt, int B, int T, int d_in,
                      int d_out, float* sqnorm_out, void* ws, size_t ws_bytes, void* stream) {
  dp_layer ly;
  ly.a = a;
  ly.g = g;
  ly.T = T;
  ly.d_in = d_in;
  ly.d_out = d_out;
  ly.path = path;
  return norms_impl(&ly, 1, dt, B, sqnorm_out, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

}  // namespace

extern "C" {

const char* dp_status_string(dp_status s) {
  switch (s) {
    case DP_OK: return "ok";
    case DP_ERR_INVALID_ARG: return "invalid argument";
    case DP_ERR_UNSUPPORTED: return "unsupported";
    case DP_ERR_WORKSPACE: return "workspace missing or too small";
    case DP_ERR_HIP: return "HIP runtime error";
  }
  return "unknown status";
}

int dp_version(void) { return 100; }

dp_path dp_choose_path(int64_t T, int64_t d_in, int64_t d_out) {
  if (T <= 0 || d_in <= 0 || d_out <= 0) return DP_PATH_GHOST;
  // 2 T^2 <= d_in d_out without overflow: compare in 128 bits.
  const __int128 lhs = (__int128)2 * T * T, rhs = (__int128)d_in * d_out;
  return lhs <= rhs ? DP_PATH_GHOST : DP_PATH_PEREX;
}

size_t dp_norm_workspace_bytes(dp_path path, dp_dtype dt, int B, int T, int d_in, int d_out) {
  dp_layer ly = {nullptr, nullptr, T, d_in, d_out, (int32_t)path};
  return dp_norms_multi_workspace_bytes(&ly, 1, dt, B);
}

size_t dp_norms_multi_workspace_bytes(const dp_layer* layers, int L, dp_dtype dt, int B) {
  if (!dtype_ok(dt)) return 0;
  const int64_t slots = norm_slots(layers, L, dt, B, nullptr);
  if (slots < 0) return 0;
  // never 0 for a valid request, so "0 = invalid" stays unambiguous
  return (size_t)(slots > 0 ? slots : 4) * sizeof(float);
}

dp_status dp_ghost_norm(const void* a, const void* g, dp_dtype dt, int B, int T, int d_in, int d_out,
                        float* sqnorm_out, void* ws, size_t ws_bytes, void* stream) {
  return single_norm(DP_PATH_GHOST, a, g, dt, B, T, d_in, d_out, sqnorm_out, ws, ws_bytes, stream);
}

dp_status dp_perex_norm(const void* a, const void* g, dp_dtype dt, int B, int T, int d_in, int d_out,
                        float* sqnorm_out, void* ws, size_t ws_bytes, void* stream) {
  return single_norm(DP_PATH_PEREX, a, g, dt, B, T, d_in, d_out, sqnorm_out, ws, ws_bytes, stream);
}

dp_status dp_norms_multi(const dp_layer* layers, int L, dp_dtype dt, int B, float* sqnorm_out, void* ws,
                         size_t ws_bytes, void* stream) {
  return norms_impl(layers, L, dt, B, sqnorm_out, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

dp_status dp_clip_factors(const float* sqnorm, int L, int B, dp_clip_mode mode, float R, float stability,
                          float* C_out, float* norm_out, void* stream) {
  if (!sqnorm || !C_out || L <= 0 || B <= 0) return DP_ERR_INVALID_ARG;
  if (mode != DP_CLIP_STANDARD && mode != DP_CLIP_AUTOMATIC) return DP_ERR_INVALID_ARG;
  if (!(R > 0.f)) return DP_ERR_INVALID_ARG;                      // rejects NaN too
  if (!(stability >= 0.f) || isinf(stability)) return DP_ERR_INVALID_ARG;
  return launch_clip_factors(sqnorm, L, B, (int)mode, R, stability, C_out, norm_out,
                             static_cast<hipStream_t>(stream));
}

}  // extern "C"

namespace {

// Clip-weighted gradients of a stack; layer l uses the weights C[c_off[l] + i] (c_off == nullptr:
// every layer uses C[i]).
// Noise request of dp_clipped_grad_noise_multi, validated.
struct NoiseSpec {
  const uint64_t* grad_offset;   // host, [L]
  uint64_t lo, hi;               // global element range that receives noise
  float stddev;
  uint64_t seed, step;
};

// Everything of a kernel's noise arguments but the layers' offsets.
void set_noise(NoiseArgs& na, const NoiseSpec& noise) {
  na.stddev = noise.stddev;
  na.step_lo = (uint32_t)noise.step;
  na.step_hi = (uint32_t)(noise.step >> 32);
  na.lo = noise.lo;
  na.hi = noise.hi;
  na.rk = make_round_keys(noise.seed);
}

// Separate noise pass on the part of layer l's gradient that lies inside the range.
dp_status noise_after(const NoiseSpec* noise, int l, const dp_layer& ly, float* grad, hipStream_t s) {
  if (!noise) return DP_OK;
  const uint64_t begin = noise->grad_offset[l], end = begin + (uint64_t)ly.d_in * ly.d_out;
  const uint64_t lo = std::max(begin, noise->lo), hi = std::min(end, noise->hi);
  if (lo >= hi) return DP_OK;
  return launch_noise(grad + (lo - begin), lo, hi - lo, noise->stddev, noise->seed, noise->step, s);
}

// Which gradient kernel a 16-bit layer takes.
//  kGradPacked: short samples.  The large-tile kernels (256 x 256, 128 x 128) pay per sample, ~600 clocks and ~700 per
//    begun 16 tokens; the packed one pays per row, three matrix instructions (fp16: six) where they need one, but its
//    tiles cover a narrow side without padding, and its error against 64 bits is smaller.  Gradients, us and relative
//    error (48 layers 1024 x side, 16384 rows; 128 and more: eight layers 1024 x 1024 .. 4096, 4096 rows):
//      sides           packed below   packed          128 x 128 or larger tiles
//      up to 32        fp16 48        575, 8.1e-7     823 at T = 16, 529 at 28, 532 at 48; 9 to 11e-7
//      33 .. 64        fp16 28        810, 8.1e-7     1312 at T = 10, 827 at 16, 732 at 20, 539 at 28; 10 to 13e-7
//      65 .. 127       bf16 48        630, 8.1e-7     830 at T = 16, 730 at 20, 616 at 24, 507 at 32, 539 at 48; 9 to 11e-7
//                      fp16 18        1214, 8.1e-7    1640 at T = 8, 1099 at 12, 833 at 16; 10 to 13e-7
//      128 and more    bf16 20        470, 4.0e-7     645 at T = 8, 443 at 12, 339 at 16, 310 at 20; 5 to 8e-7
//                      fp16 10        910, 4.0e-7     1261 at T = 4, 850 at 6, 645 at 8, 524 at 10; 6 to 14e-7
//    The lines are where the times met while the tiles padded a sample to 32 rows.  With 16-row k-steps the tiles are the
//    faster ones from fewer tokens on, but a size that has had the packed kernel's accuracy keeps it.
//    A batch of one or two samples pays the other kernels next to nothing: eight layers 4096 x 4096, one token: 141 us
//    packed, 129 on the tiles (fp16 158 and 131), one layer 72 x 3000 12.5 and 7.1, 24 layers 768 x 3072 64 and 60.
//    In fp16, sides up to 64 stay packed below 1024 rows of the batch, where the tiles' padding of the side is not paid
//    for yet: seven layers 6016 x 64, 40 rows 11 us and 20, 918 rows 49 and 70, 1024 rows 53 and 49.
//    (A layer's kernel depends on nothing but the layer and the batch: the same bits in any stack.)
//  kGradBig: slabs its 32-bit addressing reaches.
//  kGradEdge: the rest.
enum GradKernel { kGradBig = 0, kGradPacked = 1, kGradEdge = 2 };
constexpr int kGradKernels = 3;

// Samples of fewer tokens than this take the packed kernel.
int packed_below(int side, bool f16, int64_t rows) {
  if (side <= 64 && (!f16 || rows < 1024)) return INT32_MAX;
  if (side <= 32) return 48;
  if (side <= 64) return 28;
  if (side < 128) return f16 ? 18 : 48;
  return f16 ? 10 : 20;
}

GradKernel grad_kernel_of(const dp_layer& ly, dp_dtype dt, int B) {
  const int side = std::min(ly.d_in, ly.d_out);
  const bool few = side > 64 && B <= 2;
  const bool packed = !few && ly.T < packed_below(side, dt == DP_F16, (int64_t)B * ly.T);
  if (packed && grad_packed_supports(B, ly.T, ly.d_in, ly.d_out)) return kGradPacked;
  return clipped_grad_big_supports(ly.T, ly.d_in, ly.d_out) ? kGradBig : kGradEdge;
}

// What the gradient calls refuse of a layer whose a and g they read.
dp_status check_grad_layer(const dp_layer& ly, dp_dtype dt, int B, const float* grad) {
  if (!dims_ok(dt, B, ly.T, ly.d_in, ly.d_out)) return DP_ERR_INVALID_ARG;
  const dp_status st = check_layer_ptrs(ly.a, ly.g);
  if (st != DP_OK) return st;
  if (!grad || !aligned16(grad)) return DP_ERR_INVALID_ARG;
  const int64_t tiles = dt == DP_F32 ? clipped_grad_f32_tiles(ly.d_in, ly.d_out) : clipped_grad_tiles(ly.d_in, ly.d_out);
  return tiles > INT32_MAX / 2 ? DP_ERR_INVALID_ARG : DP_OK;              // one layer beyond the grid's range
}

// Everything that launch_grads' callers refuse (but for the noise: make_noise).  out16: grads[l] address 16-bit arrays of
// the operands' storage type; only the large-tile kernels write those, with the noise in their epilogue, so every layer
// must qualify for them.
dp_status check_grads(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C, float* const* grads,
                      int accumulate, const NoiseSpec* noise = nullptr, bool out16 = false) {
  if (!dtype_ok(dt)) return DP_ERR_INVALID_ARG;
  if (!layers || !grads || !C || L <= 0 || B <= 0) return DP_ERR_INVALID_ARG;
  if (accumulate != 0 && accumulate != 1) return DP_ERR_INVALID_ARG;
  for (int l = 0; l < L; ++l) {
    const dp_status st = check_grad_layer(layers[l], dt, B, grads[l]);
    if (st != DP_OK) return st;
  }
  if (!out16) return DP_OK;
  if (dt == DP_F32) return DP_ERR_UNSUPPORTED;
  for (int l = 0; l < L; ++l) {
    const dp_layer& ly = layers[l];
    if (!(ly.T % 32 == 0 && ly.d_in >= 128 && ly.d_out >= 128 && clipped_grad_big_supports(ly.T, ly.d_in, ly.d_out)))
      return DP_ERR_UNSUPPORTED;
    if (noise && (noise->grad_offset[l] & 3)) return DP_ERR_UNSUPPORTED;
  }
  return DP_OK;
}

// Noise arguments as the caller gave them.  *noisy: there is some to add; *spec is filled then.
dp_status make_noise(const dp_layer* layers, int L, const uint64_t* grad_offset, uint64_t shard_offset,
                     uint64_t shard_count, float sigma, float R, uint64_t seed, uint64_t step, NoiseSpec* spec, bool* noisy) {
  if (!(sigma >= 0.f) || isinf(sigma)) return DP_ERR_INVALID_ARG;
  if (!(R > 0.f)) return DP_ERR_INVALID_ARG;
  if (shard_offset + shard_count < shard_offset) return DP_ERR_INVALID_ARG;   // wraps 2^64
  *noisy = sigma > 0.f && shard_count > 0;
  if (!*noisy) return DP_OK;
  if (isinf(R) || !grad_offset || !layers || L <= 0) return DP_ERR_INVALID_ARG;
  for (int l = 0; l < L; ++l) {
    const uint64_t n = (uint64_t)std::max(layers[l].d_in, 0) * (uint64_t)std::max(layers[l].d_out, 0);
    if (grad_offset[l] + n < grad_offset[l]) return DP_ERR_INVALID_ARG;
  }
  spec->grad_offset = grad_offset;
  spec->lo = shard_offset;
  spec->hi = shard_offset + shard_count;
  spec->stddev = sigma * R;
  spec->seed = seed;
  spec->step = step;
  return DP_OK;
}

// Whether a layer's rows leave the matrix-core gradient kernels by streaming stores, past the caches; in a call that writes `bytes`,
// round_bytes of them in each of a launch's `rounds` of 256 large tiles.  Streaming to cached, ratios of times (3200 measurements,
// groups of them): up to 32 MB, what the L2s hold together, 0.93 to 1.02, also with a pass behind it that reads the gradient.  Beyond it
//  * without noise a gradient is there to be read again (by the noise, the next micro-batch, a reduction), and the memory-side cache
//    holds it up to some 200 MB: alone 0.99 to 1.00, with what reads it 1.01 to 1.07; above 0.94 to 1.02;
//  * rows that are not whole 128-byte lines: the two pieces of a line meet in L2 only if they stay there.  Without noise 1.01 to
//    1.13 (2 x 32 tokens, 39 layers 1016 x 1016 1.61); with noise short contractions wait for the stores, the longer the more
//    the compute units store at once: 128 to 384 rows 0.96 to 1.35; steps of 576 rows and more 0.83 to 1.02 in rounds of up to 44 MB (few
//    or ragged tiles), in fuller ones 1.02 to 1.15 of 640 and 768 rows, of 1024 to 1536 rows 1.01 to 1.12 of a single round and 0.92 to 1.01 of
//    more; from 2048 rows on 0.85 to 1.04; of calls that no cache holds, above 256 MB, 0.82 to 1.07 but for 64 rows, 0.81 to 1.30;
//  * packed rows, which take longer for what they write: above 256 MB 0.84 to 1.11, on average 0.97; below, rows of no whole lines with
//    noise 0.93 to 1.06, of 64 rows 1.01 to 1.34;
//  * whole lines with noise 0.94 to 1.02.
// An accumulating launch has just read what it writes: 1.00 either way, cached.
bool rows_stream(const GroupLayer& ly, int B, bool packed, int64_t bytes, double round_bytes, double rounds, bool noise, bool out16) {
  constexpr int64_t kInL2 = 32 << 20, kPartOfARound = 44 << 20, kInMemorySideCache = 200 << 20, kInNone = 256 << 20;
  const bool whole_lines = ly.d_out % (out16 ? 64 : 32) == 0 && reinterpret_cast<uintptr_t>(ly.out) % 128 == 0;
  if (bytes <= kInL2 || (packed && bytes > kInNone)) return true;
  if (!noise) return whole_lines && bytes > kInMemorySideCache;
  const int short_rows = packed || bytes > kInNone ? 128 : round_bytes <= kPartOfARound ? 512 : rounds < 1.4 ? 1536 : 768;
  return whole_lines || (int64_t)B * ly.T > short_rows;
}

// The gradient kernels of layers that check_grads has passed.
dp_status launch_grads(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C, const int* c_off,
                       float* const* grads, int accumulate, hipStream_t s, const NoiseSpec* noise = nullptr,
                       bool out16 = false) {
  if (dt == DP_F32) {
    NoiseArgs na = {};
    if (noise) set_noise(na, *noise);
    int l = 0;
    while (l < L) {
      GroupArgs ga;
      ga.B = B;
      ga.accumulate = accumulate;
      ga.f16 = 0;
      ga.n_layers = 0;
      int64_t blocks = 0;
      for (; l < L && ga.n_layers < kMaxGroup; ++l) {
        const int64_t tiles = clipped_grad_f32_tiles(layers[l].d_in, layers[l].d_out);
        if (ga.n_layers > 0 && blocks + tiles > INT32_MAX / 2) break;
        if (noise) na.layer_off[ga.n_layers] = noise->grad_offset[l];
        GroupLayer& gl = ga.layer[ga.n_layers++];
        gl = {};
        gl.a = layers[l].a;
        gl.g = layers[l].g;
        gl.out = grads[l];
        gl.T = layers[l].T;
        gl.d_in = layers[l].d_in;
        gl.d_out = layers[l].d_out;
        gl.tile_begin = (int)blocks;
        gl.c_off = c_off ? c_off[l] : 0;
        blocks += tiles;
      }
      ga.total_blocks = (int)blocks;
      dp_status st = launch_clipped_grad_f32_group(ga, C, na, s);
      if (st != DP_OK) return st;
    }
    return DP_OK;
  }
  std::vector<int> of_kernel[kGradKernels];
  int64_t bytes = 0;                                     // of the call
  auto grad_bytes = [&](int d, int p) { return (int64_t)d * p * (out16 ? 2 : 4); };
  for (int l = 0; l < L; ++l) {
    of_kernel[grad_kernel_of(layers[l], dt, B)].push_back(l);
    bytes += grad_bytes(layers[l].d_in, layers[l].d_out);
  }
  for (int kernel = 0; kernel < kGradKernels; ++kernel) {
    const std::vector<int>& which = of_kernel[kernel];
    size_t pos = 0;
    while (pos < which.size()) {
      GroupArgs ga;
      ga.B = B;
      ga.accumulate = accumulate;
      ga.f16 = dt == DP_F16;
      ga.n_layers = 0;
      int64_t blocks = 0;
      while (pos < which.size() && ga.n_layers < kMaxGroup) {
        const int l = which[pos];
        const int d = layers[l].d_in, p = layers[l].d_out;
        const int64_t tiles = kernel == kGradBig      ? clipped_grad_big_tiles(d, p)
                              : kernel == kGradPacked ? grad_packed_tiles(d, p)
                                                      : clipped_grad_tiles(d, p);
        if (ga.n_layers > 0 && blocks + tiles > INT32_MAX / 2) break;
        GroupLayer& gl = ga.layer[ga.n_layers++];
        gl.a = layers[l].a;
        gl.g = layers[l].g;
        gl.out = grads[l];
        gl.T = layers[l].T;
        gl.d_in = d;
        gl.d_out = p;
        gl.path = kernel == kGradPacked ? grad_packed_shape(d, p) : 0;
        gl.tile_begin = (int)blocks;
        gl.sq_index = l;
        gl.part_begin = 0;
        gl.tiles_per_sample = (int)tiles;
        gl.c_off = c_off ? c_off[l] : 0;
        blocks += tiles;
        ++pos;
      }
      ga.total_blocks = (int)blocks;
      // The kernels add the noise in their epilogue when every layer of the launch starts on a
      // generator block (offset a multiple of 4); otherwise, and for the 64-bit fallback, the noise
      // pass runs on the layer's slice afterwards.
      bool fused = noise && kernel != kGradEdge;
      NoiseArgs na;
      if (fused) {
        for (int j = 0; j < ga.n_layers; ++j) {
          na.layer_off[j] = noise->grad_offset[ga.layer[j].sq_index];
          fused = fused && (na.layer_off[j] & 3) == 0;
        }
      }
      if (fused) set_noise(na, *noise);
      const NoiseArgs* in_kernel = fused ? &na : nullptr;
      int64_t launch_bytes = 0;
      for (int j = 0; j < ga.n_layers; ++j) launch_bytes += grad_bytes(ga.layer[j].d_in, ga.layer[j].d_out);
      const double rounds = std::max(1.0, (kernel == kGradBig ? (double)blocks : launch_bytes / 262144.0) / 256);
      for (int j = 0; j < ga.n_layers; ++j)
        ga.layer[j].stream = !accumulate && rows_stream(ga.layer[j], B, kernel == kGradPacked, bytes, launch_bytes / rounds, rounds, fused, out16);
      dp_status st = kernel == kGradBig      ? launch_clipped_grad_big_group(ga, C, in_kernel, s, out16)
                     : kernel == kGradPacked ? launch_grad_packed_group(ga, C, in_kernel, s)
                                             : launch_clipped_grad_group(ga, C, s);
      if (st != DP_OK) return st;
      if (noise && !fused) {
        for (int j = 0; j < ga.n_layers; ++j) {
          const int l = ga.layer[j].sq_index;
          st = noise_after(noise, l, layers[l], grads[l], s);
          if (st != DP_OK) return st;
        }
      }
    }
  }
  return DP_OK;
}

dp_status clipped_grad_impl(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C, const int* c_off,
                            float* const* grads, int accumulate, void* stream, const NoiseSpec* noise = nullptr,
                            bool out16 = false) {
  const dp_status st = check_grads(layers, L, dt, B, C, grads, accumulate, noise, out16);
  if (st != DP_OK) return st;
  return launch_grads(layers, L, dt, B, C, c_off, grads, accumulate, static_cast<hipStream_t>(stream), noise, out16);
}

// Sum_i C_i G_i from kept per-sample gradients for the layers that have them (kept[l] != nullptr),
// up to kMaxGroup layers per launch.  c_off (or nullptr): layer l's weights are C[c_off[l] + i].
// noise (or nullptr): added by the same kernel when the layer starts on a generator block, else
// by a pass afterwards.
dp_status kept_sum_impl(const dp_layer* layers, int L, int B, const float* C, const int* c_off,
                        float* const* kept, float* const* grads, const NoiseSpec* noise, int accumulate,
                        hipStream_t s) {
  const bool noisy = noise != nullptr && noise->stddev > 0.f;
  NoiseArgs na = {};
  if (noisy) set_noise(na, *noise);
  int l = 0;
  while (l < L) {
    GroupArgs ga;
    ga.B = B;
    ga.accumulate = accumulate;
    ga.f16 = 0;
    ga.n_layers = 0;
    int64_t blocks = 0;
    int members[kMaxGroup];
    for (; l < L && ga.n_layers < kMaxGroup; ++l) {
      if (!kept || !kept[l]) continue;
      const int nb = kept_blocks(layers[l].d_in, layers[l].d_out);
      if (ga.n_layers > 0 && blocks + nb > INT32_MAX / 2) break;
      GroupLayer& gl = ga.layer[ga.n_layers];
      gl.a = kept[l];
      gl.g = nullptr;
      gl.out = grads[l];
      gl.T = layers[l].T;
      gl.d_in = layers[l].d_in;
      gl.d_out = layers[l].d_out;
      gl.path = DP_PATH_PEREX;
      gl.tile_begin = (int)blocks;
      gl.sq_index = l;
      gl.part_begin = 0;
      gl.tiles_per_sample = nb;
      gl.c_off = c_off ? c_off[l] : 0;
      na.layer_off[ga.n_layers] =
          noisy && (noise->grad_offset[l] & 3) == 0 ? noise->grad_offset[l] : ~(uint64_t)0;
      members[ga.n_layers] = l;
      blocks += nb;
      ++ga.n_layers;
    }
    if (ga.n_layers == 0) break;
    ga.total_blocks = (int)blocks;
    dp_status st = launch_kept_weighted_sum(ga, C, na, s);
    if (st != DP_OK) return st;
    for (int j = 0; j < ga.n_layers; ++j)
      if (noisy && na.layer_off[j] == ~(uint64_t)0) {
        st = noise_after(noise, members[j], layers[members[j]], grads[members[j]], s);
        if (st != DP_OK) return st;
      }
  }
  return DP_OK;
}

}  // namespace

extern "C" {

dp_status dp_clipped_grad_multi(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C,
                                float* const* grads, int accumulate, void* stream) {
  return clipped_grad_impl(layers, L, dt, B, C, nullptr, grads, accumulate, stream);
}

dp_status dp_clipped_grad_noise_multi(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C,
                                      float* const* grads, const uint64_t* grad_offset, int accumulate,
                                      uint64_t shard_offset, uint64_t shard_count, float sigma, float R,
                                      uint64_t seed, uint64_t step, void* stream) {
  NoiseSpec spec;
  bool noisy;
  const dp_status st = make_noise(layers, L, grad_offset, shard_offset, shard_count, sigma, R, seed, step, &spec, &noisy);
  if (st != DP_OK) return st;
  return clipped_grad_impl(layers, L, dt, B, C, nullptr, grads, accumulate, stream, noisy ? &spec : nullptr);
}

dp_status dp_clipped_grad_noise_multi_h16(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C,
                                          void* const* grads16, const uint64_t* grad_offset, int accumulate,
                                          uint64_t shard_offset, uint64_t shard_count, float sigma, float R,
                                          uint64_t seed, uint64_t step, void* stream) {
  NoiseSpec spec;
  bool noisy;
  const dp_status st = make_noise(layers, L, grad_offset, shard_offset, shard_count, sigma, R, seed, step, &spec, &noisy);
  if (st != DP_OK) return st;
  float* const* grads = reinterpret_cast<float* const*>(grads16);      // the kernels store 16-bit values there
  return clipped_grad_impl(layers, L, dt, B, C, nullptr, grads, accumulate, stream, noisy ? &spec : nullptr, true);
}

dp_status dp_clipped_grad_grouped(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C,
                                  const int32_t* group_of_layer, int M, float* const* grads,
                                  int accumulate, void* stream) {
  if (!group_of_layer || L <= 0 || M <= 0 || B <= 0 || (int64_t)M * B > INT32_MAX) return DP_ERR_INVALID_ARG;
  std::vector<int> c_off(L);
  for (int l = 0; l < L; ++l) {
    if (group_of_layer[l] < 0 || group_of_layer[l] >= M) return DP_ERR_INVALID_ARG;
    c_off[l] = group_of_layer[l] * B;
  }
  return clipped_grad_impl(layers, L, dt, B, C, c_off.data(), grads, accumulate, stream);
}

dp_status dp_clip_factors_grouped(const float* sqnorm, int L, int B, const int32_t* group_begin, int M,
                                  const float* R, dp_clip_mode mode, float stability, float* C_out,
                                  float* norm_out, void* stream) {
  if (!sqnorm || !C_out || !group_begin || !R || L <= 0 || B <= 0 || M <= 0) return DP_ERR_INVALID_ARG;
  if (mode != DP_CLIP_STANDARD && mode != DP_CLIP_AUTOMATIC) return DP_ERR_INVALID_ARG;
  if (!(stability >= 0.f) || isinf(stability)) return DP_ERR_INVALID_ARG;
  if (group_begin[0] != 0 || group_begin[M] != L) return DP_ERR_INVALID_ARG;
  for (int m = 0; m < M; ++m) {
    if (group_begin[m + 1] < group_begin[m]) return DP_ERR_INVALID_ARG;     // empty groups are allowed
    if (!(R[m] > 0.f)) return DP_ERR_INVALID_ARG;
  }
  return launch_clip_factors_grouped(sqnorm, B, group_begin, M, R, (int)mode, stability, C_out, norm_out,
                                     static_cast<hipStream_t>(stream));
}

float dp_group_noise_threshold(const float* R, int M) {
  if (!R || M <= 0) return 0.f;
  double s = 0.0;
  for (int m = 0; m < M; ++m) s += (double)R[m] * R[m];
  return (float)sqrt(s);
}

dp_status dp_bias_norm(const void* g, dp_dtype dt, int B, int T, int d_out, float* colsum,
                       float* sqnorm_out, void* stream) {
  if (!dtype_ok(dt)) return DP_ERR_INVALID_ARG;
  if (!g || !colsum || !sqnorm_out || !aligned16(g)) return DP_ERR_INVALID_ARG;
  if (!dims_ok(dt, B, T, 8, d_out)) return DP_ERR_INVALID_ARG;
  if (B > 65535) return DP_ERR_UNSUPPORTED;
  return launch_bias_norm(g, dt, B, T, d_out, colsum, sqnorm_out, static_cast<hipStream_t>(stream));
}

dp_status dp_clipped_bias_grad(const float* colsum, int B, int d_out, const float* C, float* grad_b,
                               int accumulate, void* stream) {
  if (!colsum || !C || !grad_b || B <= 0 || d_out <= 0) return DP_ERR_INVALID_ARG;
  if (accumulate != 0 && accumulate != 1) return DP_ERR_INVALID_ARG;
  return launch_clipped_bias_grad(colsum, B, d_out, C, grad_b, accumulate, static_cast<hipStream_t>(stream));
}

dp_status dp_clipped_grad(const void* a, const void* g, dp_dtype dt, int B, int T, int d_in, int d_out,
                          const float* C, float* grad, int accumulate, void* stream) {
  dp_layer ly = {a, g, T, d_in, d_out, 0};
  float* grads[1] = {grad};
  return dp_clipped_grad_multi(&ly, 1, dt, B, C, grads, accumulate, stream);
}

dp_status dp_add_noise(float* grad_slice, uint64_t global_offset, uint64_t count, float sigma, float R,
                       uint64_t seed, uint64_t step, void* stream) {
  if (!(sigma >= 0.f) || isinf(sigma)) return DP_ERR_INVALID_ARG;
  if (!(R > 0.f)) return DP_ERR_INVALID_ARG;
  if (global_offset + count < global_offset) return DP_ERR_INVALID_ARG;   // wraps 2^64
  if (sigma == 0.f || count == 0) return DP_OK;                            // non-private: nothing to add
  if (isinf(R)) return DP_ERR_INVALID_ARG;
  if (!grad_slice || (reinterpret_cast<uintptr_t>(grad_slice) & 3u)) return DP_ERR_INVALID_ARG;
  return launch_noise(grad_slice, global_offset, count, sigma * R, seed, step,
                      static_cast<hipStream_t>(stream));
}

dp_status dp_philox_blocks(uint32_t* out, uint64_t first_block, uint64_t n_blocks, uint64_t seed,
                           uint64_t step, void* stream) {
  if (!out || !aligned16(out)) return DP_ERR_INVALID_ARG;
  if (n_blocks == 0) return DP_OK;
  if (first_block + n_blocks < first_block) return DP_ERR_INVALID_ARG;
  return launch_philox_blocks(out, first_block, n_blocks, seed, step, static_cast<hipStream_t>(stream));
}

}  // extern "C"


// ---------------------------------------------------------------------------------
// Instantiated layers with their per-sample gradients kept between the two halves.
// ---------------------------------------------------------------------------------
namespace {

// kept[l] may be given only for 16-bit layers on the instantiated path, 16-byte aligned.
dp_status check_kept(const dp_layer* layers, int L, dp_dtype dt, float* const* kept) {
  if (!kept) return DP_OK;
  for (int l = 0; l < L; ++l) {
    if (!kept[l]) continue;
    if (dt == DP_F32) return DP_ERR_UNSUPPORTED;
    if (layers[l].path != DP_PATH_PEREX || !aligned16(kept[l])) return DP_ERR_INVALID_ARG;
    if ((int64_t)layers[l].d_in * layers[l].d_out > INT32_MAX - 4096) return DP_ERR_INVALID_ARG;   // int element index
  }
  return DP_OK;
}

// Everything that launch_grads_kept's callers refuse, but for the noise.
dp_status check_grads_kept(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C, float* const* kept,
                           float* const* grads, int accumulate) {
  if (!layers || !grads || !C || L <= 0 || B <= 0 || !dtype_ok(dt)) return DP_ERR_INVALID_ARG;
  if (accumulate != 0 && accumulate != 1) return DP_ERR_INVALID_ARG;
  for (int l = 0; l < L; ++l) {
    if (!dims_ok(dt, B, layers[l].T, layers[l].d_in, layers[l].d_out)) return DP_ERR_INVALID_ARG;
    if (layers[l].path != DP_PATH_GHOST && layers[l].path != DP_PATH_PEREX) return DP_ERR_INVALID_ARG;
    if (!grads[l] || !aligned16(grads[l])) return DP_ERR_INVALID_ARG;
  }
  dp_status st = check_kept(layers, L, dt, kept);
  for (int l = 0; l < L && st == DP_OK; ++l)
    if (!kept || !kept[l]) st = check_grad_layer(layers[l], dt, B, grads[l]);
  return st;
}

// Layers without kept gradients: the contraction over a and g; with: weighted sums.
dp_status launch_grads_kept(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C, float* const* kept,
                            float* const* grads, int accumulate, hipStream_t s, const NoiseSpec* noise) {
  std::vector<dp_layer> sub;
  std::vector<float*> sub_grads;
  std::vector<uint64_t> sub_off;
  for (int l = 0; l < L; ++l)
    if (!kept || !kept[l]) {
      sub.push_back(layers[l]);
      sub_grads.push_back(grads[l]);
      sub_off.push_back(noise ? noise->grad_offset[l] : 0);
    }
  if (!sub.empty()) {
    NoiseSpec sub_spec;
    if (noise) sub_spec = *noise;
    sub_spec.grad_offset = sub_off.data();
    const dp_status st = launch_grads(sub.data(), (int)sub.size(), dt, B, C, nullptr, sub_grads.data(), accumulate, s,
                                      noise ? &sub_spec : nullptr);
    if (st != DP_OK) return st;
  }
  return kept_sum_impl(layers, L, B, C, nullptr, kept, grads, noise, accumulate, s);
}

}  // namespace

extern "C" {

dp_status dp_norms_multi_keep(const dp_layer* layers, int L, dp_dtype dt, int B, float* sqnorm_out,
                              float* const* kept, void* ws, size_t ws_bytes, void* stream) {
  if (!layers || L <= 0) return DP_ERR_INVALID_ARG;
  for (int l = 0; l < L; ++l)
    if (layers[l].path != DP_PATH_GHOST && layers[l].path != DP_PATH_PEREX) return DP_ERR_INVALID_ARG;
  dp_status st = check_kept(layers, L, dt, kept);
  if (st != DP_OK) return st;
  return norms_impl(layers, L, dt, B, sqnorm_out, ws, ws_bytes, static_cast<hipStream_t>(stream), nullptr, kept);
}

dp_status dp_clipped_grad_kept_multi(const dp_layer* layers, int L, dp_dtype dt, int B, const float* C,
                                     float* const* kept, float* const* grads, const uint64_t* grad_offset,
                                     int accumulate, uint64_t shard_offset, uint64_t shard_count, float sigma,
                                     float R, uint64_t seed, uint64_t step, void* stream) {
  NoiseSpec spec;
  bool noisy;
  dp_status st = make_noise(layers, L, grad_offset, shard_offset, shard_count, sigma, R, seed, step, &spec, &noisy);
  if (st == DP_OK) st = check_grads_kept(layers, L, dt, B, C, kept, grads, accumulate);
  if (st != DP_OK) return st;
  return launch_grads_kept(layers, L, dt, B, C, kept, grads, accumulate, static_cast<hipStream_t>(stream),
                           noisy ? &spec : nullptr);
}

dp_status dp_private_step_multi(const dp_layer* layers, int L, dp_dtype dt, int B, dp_clip_mode mode, float R,
                                float stability, float* const* kept, float* const* grads, const uint64_t* grad_offset,
                                int accumulate, uint64_t shard_offset, uint64_t shard_count, float sigma, uint64_t seed,
                                uint64_t step, float* sqnorm_out, float* C_out, float* norm_out, void* ws,
                                size_t ws_bytes, void* counter, void* stream) {
  if (!layers || L <= 0 || !C_out) return DP_ERR_INVALID_ARG;
  if (reinterpret_cast<uintptr_t>(counter) & 3u) return DP_ERR_INVALID_ARG;
  if (mode != DP_CLIP_STANDARD && mode != DP_CLIP_AUTOMATIC) return DP_ERR_INVALID_ARG;
  if (!(R > 0.f) || !(stability >= 0.f) || isinf(stability)) return DP_ERR_INVALID_ARG;
  // All that the gradients refuse before the norms, which check the rest and launch.
  NoiseSpec spec;
  bool noisy;
  dp_status st = make_noise(layers, L, grad_offset, shard_offset, shard_count, sigma, R, seed, step, &spec, &noisy);
  if (st == DP_OK)
    st = kept ? check_grads_kept(layers, L, dt, B, C_out, kept, grads, accumulate)
              : check_grads(layers, L, dt, B, C_out, grads, accumulate);
  if (st != DP_OK) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const ClipSpec clip = {(int)mode, stability, C_out, nullptr, R, norm_out, static_cast<unsigned*>(counter)};
  st = norms_impl(layers, L, dt, B, sqnorm_out, ws, ws_bytes, s, nullptr, kept, &clip);
  if (st != DP_OK) return st;
  const NoiseSpec* noise = noisy ? &spec : nullptr;
  return kept ? launch_grads_kept(layers, L, dt, B, C_out, kept, grads, accumulate, s, noise)
              : launch_grads(layers, L, dt, B, C_out, nullptr, grads, accumulate, s, noise);
}

}  // extern "C"

// ---------------------------------------------------------------------------------
// Layer-wise clipping without book-keeping (section 3.3 (II); appendix on the hook-free form).
// ---------------------------------------------------------------------------------
namespace {

// A pass ends once its a and g exceed half the memory-side cache, but not before it holds enough
// gradient tiles for four rounds of workgroups: launches that leave compute units idle cost more
// than re-reading a and g from memory (measured on a GPT-2-small stack: passes of 4 layers
// 2.3 ms, 8 layers 1.39 ms, 16 layers 1.38 ms, all norms then all gradients 1.31 ms).
constexpr int64_t kPassBytes = (int64_t)128 << 20;
constexpr int64_t kPassTiles = 1024;
// For the same reason a pass takes the rest of the stack when that would not fill two rounds (24 layers
// of width 1024, 10 x 100 fp16 tokens: a second pass of the last two layers took 83 of 347 us).
constexpr int64_t kLastPassTiles = 512;

// Which layers the one-pass kernel takes, and its sample chunks.
struct FusedPlan {
  std::vector<int> shape;        // per layer: shape class or -1
  int n_fused = 0;
  int chunks = 1;                // sample chunks per fused layer
  int64_t floats = 0;            // partial sums of all fused layers
  // Other layers on the instantiated path keep their per-sample gradients G_i between the norm and
  // the weighted sum (as dp_norms_multi_keep does): float offset of layer l's [B, d, p] block in
  // the kept region of the workspace, or -1.  Layers are taken in order while the region stays
  // within kKeptMaxBytes; the rest contract a and g a second time.
  std::vector<int64_t> kept_off;
  int64_t kept_floats = 0;
};
constexpr int64_t kKeptMaxBytes = (int64_t)2 << 30;

// The one-pass kernel saves writing and reading the per-sample gradients, but a workgroup goes through its samples one after
// the other with one k-block in flight, and it takes two launches for each shape.  Norms and factors are the same bits in
// either form, so the choice is by estimated time (us).  Steps in either form of 855 stacks of one shape or of adapter pairs, 8 to
// 4096 samples of 16 to 2048 tokens: the estimate's choice is 0.2 % above the faster one, 29 % at worst (one form for all: 17
// and 33 % above, 4 and 7.5 times as long at worst).  Fused and apart, some of them: eight layers 128 x 128, 8 x 256 tokens 14.8,
// 15.7; 8 x 2048 35.8, 24.9; 64 x 512 32.4, 40.5; 1024 x 1024 801, 1023; two of 256 x 8, 1024 x 128 52, 105, 8192 x 512
// 1101, 1620; six pairs 192 x 32, 256 x 128 131, 69; 16 of 512 x 16, 4096 x 128 1640, 2360.
bool one_pass_is_faster(const dp_layer* layers, const std::vector<int>& shape, int B, int chunks) {
  const int per = (B + chunks - 1) / chunks;
  double serial[3] = {}, longest[3] = {}, norms = 0, read_mb = 0, kept_mb = 0, room_mb = 0;
  bool others = false, kept_others = false;
  for (size_t l = 0; l < shape.size(); ++l) {
    const dp_layer& ly = layers[l];
    const double own_mb = (double)B * ly.d_in * ly.d_out * 4e-6;
    if (ly.path == DP_PATH_PEREX) room_mb += own_mb;
    if (shape[l] < 0) {
      others = true;
      kept_others = kept_others || ly.path == DP_PATH_PEREX;
      continue;
    }
    const double blocks = (ly.T + 63) / 64, chunk = per * (shape[l] == 0 ? 1.3 + 1.04 * blocks : 2.0 + 1.6 * blocks);
    longest[shape[l]] = std::max(longest[shape[l]], chunk);
    serial[shape[l]] += chunks * chunk / 256;
    norms += (double)B * perex_tiles_per_sample(ly.d_in, ly.d_out) * (3.2 + 0.0056 * ly.T) / 768;
    read_mb += (double)B * ly.T * (ly.d_in + ly.d_out) * 2e-6;
    kept_mb += own_mb;
  }
  // for each shape two launches, the second of which adds the chunks; samples one after the other, or their bytes at 6.5 TB/s
  double launches = 0, samples = 0;
  for (int k = 0; k < 3; ++k)
    if (longest[k] > 0) {
      launches += 7.4;
      samples += std::max(serial[k], longest[k]);
    }
  const double fused = launches + 0.07 * chunks + std::max(samples, read_mb / 6.5);
  // launches that no other layer needs; tiles, or bytes at 7 TB/s; the weighted sum, eight samples to a latency, or bytes at 3
  const double apart = (others ? 0 : 12.7) + std::max(norms, (read_mb + kept_mb) / 7) +
                       std::max(kept_others ? 0 : 0.094 * B, kept_mb / 3);
  return room_mb * 1e6 > kKeptMaxBytes || fused < apart;       // no room for all: some layers would be contracted twice
}

FusedPlan plan_fused(const dp_layer* layers, int L, dp_dtype dt, int B) {
  FusedPlan fp;
  fp.shape.assign(L, -1);
  fp.kept_off.assign(L, -1);
  if (dt == DP_F32) return fp;
  for (int l = 0; l < L; ++l)
    if (layers[l].path == DP_PATH_PEREX) {
      fp.shape[l] = layerwise_fused_shape(layers[l].d_in, layers[l].d_out);
      fp.n_fused += fp.shape[l] >= 0;
    }
  if (fp.n_fused > 0) {
    // enough workgroups to fill the 256 compute units when the batch allows
    const int want = std::min(B, std::max(1, 256 / fp.n_fused));
    const int per = (B + want - 1) / want;
    fp.chunks = (B + per - 1) / per;
    if (!one_pass_is_faster(layers, fp.shape, B, fp.chunks)) {
      fp.shape.assign(L, -1);
      fp.n_fused = 0;
    }
  }
  for (int l = 0; l < L; ++l) {
    const int64_t n = (int64_t)B * layers[l].d_in * layers[l].d_out;
    if (fp.shape[l] >= 0) {
      fp.floats += (int64_t)fp.chunks * layers[l].d_in * layers[l].d_out;
    } else if (layers[l].path == DP_PATH_PEREX && n <= INT32_MAX - 4096 && (fp.kept_floats + n) * 4 <= kKeptMaxBytes) {
      fp.kept_off[l] = fp.kept_floats;
      fp.kept_floats += (n + 3) & ~(int64_t)3;                    // blocks stay 16-byte aligned
    }
  }
  return fp;
}

size_t align16(size_t x) { return (x + 15) & ~(size_t)15; }

}  // namespace

extern "C" {

size_t dp_layerwise_workspace_bytes(const dp_layer* layers, int L, dp_dtype dt, int B) {
  const size_t norms = dp_norms_multi_workspace_bytes(layers, L, dt, B);
  if (norms == 0) return 0;
  const FusedPlan fp = plan_fused(layers, L, dt, B);
  if (fp.floats > INT32_MAX) return 0;
  return align16(norms) + align16((size_t)fp.floats * sizeof(float)) + (size_t)fp.kept_floats * sizeof(float);
}

dp_status dp_layerwise_clipped_grad(const dp_layer* layers, int L, dp_dtype dt, int B, const float* R,
                                    dp_clip_mode mode, float stability, float* const* grads,
                                    const uint64_t* grad_offset, int accumulate, uint64_t shard_offset,
                                    uint64_t shard_count, float sigma, uint64_t seed, uint64_t step,
                                    float* sqnorm_out, float* C_out, void* ws, size_t ws_bytes,
                                    int layers_per_pass, void* stream) {
  if (!dtype_ok(dt) || !layers || !R || !grads || !sqnorm_out || !C_out || L <= 0 || B <= 0) return DP_ERR_INVALID_ARG;
  if (mode != DP_CLIP_STANDARD && mode != DP_CLIP_AUTOMATIC) return DP_ERR_INVALID_ARG;
  if (!(stability >= 0.f) || isinf(stability)) return DP_ERR_INVALID_ARG;
  if (accumulate != 0 && accumulate != 1) return DP_ERR_INVALID_ARG;
  if (layers_per_pass < 0 || (int64_t)L * B > INT32_MAX) return DP_ERR_INVALID_ARG;
  if (!(sigma >= 0.f) || isinf(sigma)) return DP_ERR_INVALID_ARG;
  if (shard_offset + shard_count < shard_offset) return DP_ERR_INVALID_ARG;
  double r2 = 0.0;
  for (int l = 0; l < L; ++l) {
    if (!(R[l] > 0.f)) return DP_ERR_INVALID_ARG;
    r2 += (double)R[l] * R[l];
    if (!dims_ok(dt, B, layers[l].T, layers[l].d_in, layers[l].d_out)) return DP_ERR_INVALID_ARG;
    if (layers[l].path != DP_PATH_GHOST && layers[l].path != DP_PATH_PEREX) return DP_ERR_INVALID_ARG;
    dp_status st = check_layer_ptrs(layers[l].a, layers[l].g);
    if (st != DP_OK) return st;
    if (!grads[l] || !aligned16(grads[l])) return DP_ERR_INVALID_ARG;
  }
  const bool noisy = sigma > 0.f && shard_count > 0;
  const float stddev = noisy ? (float)(sigma * sqrt(r2)) : 0.f;          // eq. (1): sigma ||(R_1..R_L)||
  if (noisy) {
    if (!grad_offset || isinf(stddev)) return DP_ERR_INVALID_ARG;
    for (int l = 0; l < L; ++l) {
      const uint64_t n = (uint64_t)layers[l].d_in * (uint64_t)layers[l].d_out;
      if (grad_offset[l] + n < grad_offset[l]) return DP_ERR_INVALID_ARG;
    }
  }
  const size_t need = dp_layerwise_workspace_bytes(layers, L, dt, B);
  if (need == 0) return DP_ERR_INVALID_ARG;
  if (!ws || ws_bytes < need) return DP_ERR_WORKSPACE;
  if (!aligned16(ws)) return DP_ERR_INVALID_ARG;
  const FusedPlan fp = plan_fused(layers, L, dt, B);
  float* fused_partial = reinterpret_cast<float*>(static_cast<unsigned char*>(ws) +
                                                  align16(dp_norms_multi_workspace_bytes(layers, L, dt, B)));
  float* kept_region = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(fused_partial) +
                                                align16((size_t)fp.floats * sizeof(float)));
  hipStream_t s = static_cast<hipStream_t>(stream);

  NoiseArgs na = {};
  na.stddev = stddev;
  na.step_lo = (uint32_t)step;
  na.step_hi = (uint32_t)(step >> 32);
  na.lo = shard_offset;
  na.hi = shard_offset + shard_count;
  na.rk = make_round_keys(seed);

  auto pass_tiles = [&](int l) {
    return fp.shape[l] >= 0 ? (int64_t)0 : (int64_t)clipped_grad_big_tiles(layers[l].d_in, layers[l].d_out);
  };
  int64_t fused_off = 0, tiles_left = 0;                 // tiles of the layers from l1 on
  for (int l = 0; l < L; ++l) tiles_left += pass_tiles(l);
  for (int l0 = 0; l0 < L;) {
    // one pass: consecutive layers whose a and g stay in the memory-side cache between the norm
    // kernels and the gradient kernels (or layers_per_pass of them when the caller says so)
    int l1 = l0;
    int64_t bytes = 0, tiles = 0;
    const int64_t esize = dt == DP_F32 ? 4 : 2;
    while (l1 < L) {
      const bool small = fp.shape[l1] >= 0;
      const int64_t lb = small ? 0 : (int64_t)B * layers[l1].T * ((int64_t)layers[l1].d_in + layers[l1].d_out) * esize;
      if (l1 > l0 && (layers_per_pass > 0 ? l1 - l0 >= layers_per_pass
                                          : bytes + lb > kPassBytes && tiles >= kPassTiles &&
                                                tiles_left >= kLastPassTiles)) break;
      bytes += lb;
      tiles += pass_tiles(l1);
      tiles_left -= pass_tiles(l1);
      ++l1;
    }
    // (1) layers that fit one workgroup tile: norm, clip factor and weighted sum in one kernel
    for (int shape = 0; shape < 3; ++shape) {
      for (int l = l0; l < l1;) {
        GroupArgs ga;
        ga.B = B;
        ga.accumulate = accumulate;
        ga.f16 = dt == DP_F16;
        ga.n_layers = 0;
        float Rg[kMaxGroup];
        int blocks = 0;
        for (; l < l1 && ga.n_layers < kMaxGroup; ++l) {
          if (fp.shape[l] != shape) continue;
          GroupLayer& gl = ga.layer[ga.n_layers];
          gl.a = layers[l].a;
          gl.g = layers[l].g;
          gl.out = grads[l];
          gl.T = layers[l].T;
          gl.d_in = layers[l].d_in;
          gl.d_out = layers[l].d_out;
          gl.path = DP_PATH_PEREX;
          gl.tile_begin = blocks;
          gl.sq_index = l;
          gl.part_begin = (int)fused_off;
          gl.tiles_per_sample = fp.chunks;
          gl.c_off = 0;
          Rg[ga.n_layers] = R[l];
          na.layer_off[ga.n_layers] = noisy ? grad_offset[l] : 0;
          fused_off += (int64_t)fp.chunks * gl.d_in * gl.d_out;
          blocks += fp.chunks;
          ++ga.n_layers;
        }
        if (ga.n_layers == 0) break;
        ga.total_blocks = blocks;
        dp_status st = launch_layerwise_fused(shape, ga, Rg, (int)mode, stability, fused_partial, sqnorm_out, C_out, s);
        if (st != DP_OK) return st;
        st = launch_layerwise_reduce(ga, fused_partial, na, s);
        if (st != DP_OK) return st;
      }
    }
    // (2) the other layers of the pass: norms, clip factors, weighted gradients
    //     (instantiated layers keep G_i in the workspace: their gradient is sum_i C_i G_i)
    std::vector<dp_layer> sub;
    std::vector<int> row, c_off;
    std::vector<float> sub_R;
    std::vector<float*> sub_grads, sub_kept;
    std::vector<uint64_t> sub_off;
    bool any_kept = false;
    for (int l = l0; l < l1; ++l)
      if (fp.shape[l] < 0) {
        sub.push_back(layers[l]);
        row.push_back(l);
        sub_R.push_back(R[l]);
        c_off.push_back(l * B);
        sub_grads.push_back(grads[l]);
        sub_off.push_back(noisy ? grad_offset[l] : 0);
        sub_kept.push_back(fp.kept_off[l] >= 0 ? kept_region + fp.kept_off[l] : nullptr);
        any_kept = any_kept || fp.kept_off[l] >= 0;
      }
    if (!sub.empty()) {
      const int n = (int)sub.size();
      const ClipSpec clip = {(int)mode, stability, C_out, sub_R.data(), 0.f, nullptr, nullptr};
      dp_status st = norms_impl(sub.data(), n, dt, B, sqnorm_out, ws, ws_bytes, s, row.data(),
                                any_kept ? sub_kept.data() : nullptr, &clip);
      if (st != DP_OK) return st;
      NoiseSpec spec;
      spec.grad_offset = sub_off.data();
      spec.lo = shard_offset;
      spec.hi = shard_offset + shard_count;
      spec.stddev = stddev;
      spec.seed = seed;
      spec.step = step;
      // layers without kept gradients: the contraction over a and g
      std::vector<dp_layer> rest;
      std::vector<int> rest_c;
      std::vector<float*> rest_grads;
      std::vector<uint64_t> rest_off;
      for (int j = 0; j < n; ++j)
        if (!sub_kept[j]) {
          rest.push_back(sub[j]);
          rest_c.push_back(c_off[j]);
          rest_grads.push_back(sub_grads[j]);
          rest_off.push_back(sub_off[j]);
        }
      if (!rest.empty()) {
        NoiseSpec rest_spec = spec;
        rest_spec.grad_offset = rest_off.data();
        st = clipped_grad_impl(rest.data(), (int)rest.size(), dt, B, C_out, rest_c.data(), rest_grads.data(),
                               accumulate, stream, noisy ? &rest_spec : nullptr);
        if (st != DP_OK) return st;
      }
      if (any_kept) {
        st = kept_sum_impl(sub.data(), n, B, C_out, c_off.data(), sub_kept.data(), sub_grads.data(),
                           noisy ? &spec : nullptr, accumulate, s);
        if (st != DP_OK) return st;
      }
    }
    l0 = l1;
  }
  return DP_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------------
// dp_norms_multi for callers that cannot allocate: the per-tile partial sums go to a fixed
// array in the library's own device image instead of a caller-provided workspace.
// ---------------------------------------------------------------------------------
namespace {

constexpr size_t kStaticScratchBytes = (size_t)1 << 20;        // 262144 partial sums
constexpr int kStaticMaxLayers = 1024;

// One copy per device, at its own address; `scratch` itself is only a handle on the host side.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

std::atomic<void*> scratch_address[kMaxDevices];

// Device address of `scratch` on the current device, resolved once per device.
dp_status static_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return DP_ERR_HIP;
  void* p = scratch_address[dev].load(std::memory_order_acquire);
  if (!p) {
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DP_ERR_HIP;
    scratch_address[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return DP_OK;
}

}  // namespace

extern "C" dp_status dp_norms_multi_static(const dp_layer* layers, int L, dp_dtype dt, int B,
                                           float* sqnorm_out, void* stream) {
  if (!layers || L <= 0) return DP_ERR_INVALID_ARG;
  if (L > kStaticMaxLayers) return DP_ERR_WORKSPACE;
  const size_t need = dp_norms_multi_workspace_bytes(layers, L, dt, B);
  if (need == 0) return DP_ERR_INVALID_ARG;
  if (need > kStaticScratchBytes) return DP_ERR_WORKSPACE;
  void* ws = nullptr;
  dp_status st = static_scratch(&ws);
  if (st != DP_OK) return st;
  // Every partial sum that is read was written by this call's kernels first, so nothing in the
  // array has to start at zero.
  int64_t begin[kStaticMaxLayers];
  int idx[kNormKernels * kStaticMaxLayers];
  return norms_impl(layers, L, dt, B, sqnorm_out, ws, kStaticScratchBytes, static_cast<hipStream_t>(stream),
                    begin, idx);
}

// ---------------------------------------------------------------------------------
// Tile orders of the large-tile kernels, replayed on the host (pure functions, for tests).
// ---------------------------------------------------------------------------------
extern "C" {

dp_status dp_clipped_grad_launches(const dp_layer* layers, int n_layers, dp_dtype dt, int B, int out16, int32_t* launches) {
  if (!layers || !launches || n_layers <= 0 || (dt != DP_BF16 && dt != DP_F16)) return DP_ERR_INVALID_ARG;
  if (n_layers > kMaxGroup) return DP_ERR_UNSUPPORTED;
  GroupArgs ga = {};
  int64_t tiles = 0;
  for (int l = 0; l < n_layers; ++l) {
    const dp_layer& ly = layers[l];
    if (!dims_ok(dt, B, ly.T, ly.d_in, ly.d_out)) return DP_ERR_INVALID_ARG;
    if (grad_kernel_of(ly, dt, B) != kGradBig) return DP_ERR_UNSUPPORTED;
    GroupLayer& gl = ga.layer[l];
    gl.T = ly.T;
    gl.d_in = ly.d_in;
    gl.d_out = ly.d_out;
    tiles += clipped_grad_big_tiles(ly.d_in, ly.d_out);
    if (tiles > INT32_MAX / 2) return DP_ERR_UNSUPPORTED;
  }
  ga.n_layers = n_layers;
  ga.B = B;
  ga.total_blocks = (int)tiles;
  const GradLaunches plan = clipped_grad_launches(ga, out16 != 0);
  launches[0] = ga.total_blocks - plan.cut.tiles;
  launches[1] = plan.workgroups;
  launches[2] = plan.blocks;
  launches[3] = plan.cut.tiles;
  launches[4] = plan.cut.side;
  launches[5] = plan.cut.brief;
  return DP_OK;
}

int64_t dp_clipped_grad_tile_order(int d_in, int d_out, int32_t* tile_row0, int32_t* tile_col0,
                                   int64_t capacity) {
  if (d_in <= 0 || d_out <= 0 || capacity < 0) return -1;
  const int64_t n = clipped_grad_big_tiles(d_in, d_out);
  if (n > INT32_MAX / 2) return -1;
  // the split of a long contraction over rows of whole lines, and of up to 2048 ragged rows: the call knows neither the rows
  // nor neighbours
  const GradTail cut = clipped_grad_tail((int)n, clipped_grad_mid_tiles(d_in, d_out), INT32_MAX, true, false, false);
  const int n_main = (int)n - cut.tiles;
  const int tiles_m = (d_in + 255) / 256, tiles_n = (d_out + 255) / 256;
  auto put = [&](int64_t b, int t) {
    int tm, tn;
    grad_tile_of(tiles_m, tiles_n, t, tm, tn);
    if (tile_row0) tile_row0[b] = tm * 256;
    if (tile_col0) tile_col0[b] = tn * 256;
  };
  // workgroups of the large-tile kernel first, then the tiles that are cut, by the workgroup of their first sub-tile
  for (int b = 0; b < n_main && b < capacity; ++b) put(b, grad_logical_tile(b, n_main));
  if (capacity <= n_main) return n;
  const int subs = cut.side * cut.side;
  if ((int64_t)cut.tiles * subs > INT32_MAX) return -1;
  const int total = cut.tiles * subs;
  std::vector<uint16_t> seen(cut.tiles);
  int64_t b = n_main;
  for (int w = 0; w < total; ++w) {
    const SubTile s = cut.side == kGradTailSide ? grad_sub_tile<kGradTailSide>(w, total) : grad_sub_tile<kGradMidSide>(w, total);
    const int sub = s.row * cut.side + s.col;
    if (s.tile < 0 || s.tile >= cut.tiles || sub >= subs || (seen[s.tile] >> sub & 1)) return -1;
    seen[s.tile] |= 1 << sub;
    if (sub == 0 && b < capacity) put(b++, n_main + s.tile);
  }
  return n;
}

int64_t dp_ghost_tile_order(int T, int B, int32_t* sample, int32_t* token_row0, int32_t* token_col0,
                            int32_t* slot, int64_t capacity) {
  if (T <= 0 || B <= 0 || capacity < 0) return -1;
  const int tps = ghost_big_tiles_per_sample(T);
  const int64_t n = (int64_t)tps * B;
  if (n > INT32_MAX / 2) return -1;
  for (int64_t b = 0; b < n && b < capacity; ++b) {
    const GhostTile t = ghost_tile_of(T, tps, ghost_logical_tile((int)b, (int)n));
    if (sample) sample[b] = t.sample;
    if (token_row0) token_row0[b] = t.I * 256;
    if (token_col0) token_col0[b] = t.J * 128;
    if (slot) slot[b] = t.slot;
  }
  return n;
}

}  // extern "C"
