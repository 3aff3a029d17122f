// Clip factors (section 2.1 of the paper) as the kernels that finish a norm form them.
#pragma once

#include "dp_internal.h"

namespace dpbk {

// Norm from a sum of squared norms: rounding may have left it slightly negative.
__device__ __forceinline__ float norm_of(float total) {
  return total != total ? total : __builtin_sqrtf(fmaxf(total, 0.f));   // fmaxf drops a NaN
}

// Clip factor of one (sample, group) from its norm (section 2.1).  A NaN norm gives a NaN
// factor, so a sample whose gradient is not a number shows in the result instead of passing
// unclipped (fminf would drop the NaN).  Automatic clipping with norm + stability == 0 (a zero
// gradient and no stability constant) gives 0 rather than R/0: the sample adds nothing under any
// weight, and an infinite weight would turn its zero gradient into NaN.
__device__ __forceinline__ float clip_factor(float norm, int mode, float R, float stability) {
  if (norm != norm) return norm;
  if (mode == DP_CLIP_STANDARD) return fminf(R / norm, 1.f);     // norm == 0: R/0 = +inf -> 1
  const float den = norm + stability;
  return den > 0.f ? R / den : 0.f;
}

// Squared norm of sample i of the launch's layer l, and with layer-wise clipping the sample's factor.
__device__ __forceinline__ void store_norm(const GroupArgs& ga, const LayerClip& lc, int l, int i, float sq,
                                           float* __restrict__ sqnorm) {
  const size_t o = (size_t)ga.layer[l].sq_index * ga.B + i;
  sqnorm[o] = sq;
  if (lc.C_out) lc.C_out[o] = clip_factor(norm_of(sq), lc.mode, lc.R[l], lc.stability);
}

}  // namespace dpbk
