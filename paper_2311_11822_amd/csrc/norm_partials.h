// Squared norm of one sample of a layer from its per-tile partial sums.
#pragma once

#include "dp_internal.h"

namespace dpbk {

// By `width` neighbouring lanes (a power of two; 64, or no fewer than the layer has partial sums), of which this is lane
// `lane`: each adds a strided subset in order, then a fixed butterfly: deterministic, and the same bits at
// any width.  Four loads at a time: one after the other, 1012 sums took 1.7 us longer.
__device__ __forceinline__ float partial_sum(const GroupLayer& ly, int i, const float* __restrict__ partials, int lane,
                                             int width) {
  const float* src = partials + ly.part_begin + (size_t)i * ly.tiles_per_sample;
  float s = 0.f;
  const int n = ly.tiles_per_sample;
  for (unsigned q0 = lane; q0 < (unsigned)n; q0 += 256) {
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = q0 + 64 * j < (unsigned)n ? src[q0 + 64 * j] : 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) s += v[j];
  }
  for (int off = width / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
  return s;
}

}  // namespace dpbk
