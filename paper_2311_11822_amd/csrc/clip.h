// Clip factors (section 2.1 of the paper) as the kernels that finish a norm form them.
#pragma once

#include <type_traits>

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

// Sum of rows [l0, l1) of sqnorm at column i, by one wave: each lane adds a strided subset in
// order, then a fixed butterfly, so the result is deterministic; the rows are loaded in
// parallel (a serial loop would pay one memory latency per layer).
__device__ __forceinline__ float column_sum(const float* sqnorm, int B, int i, int l0, int l1, int lane) {
  float total = 0.f;
  for (int l = l0 + lane; l < l1; l += 64) total += sqnorm[(size_t)l * B + i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off);
  return total;
}

// Squared norm of sample i of the launch's layer l, and with layer-wise clipping the sample's factor.
__device__ __forceinline__ void store_norm(const GroupArgs& ga, const NormClip& nc, int l, int i, float sq, float* sqnorm) {
  const size_t o = (size_t)ga.layer[l].sq_index * ga.B + i;
  if (nc.kind == kGroupFactors)
    __hip_atomic_store(&sqnorm[o], sq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // read by another workgroup
  else
    sqnorm[o] = sq;
  if (nc.kind == kLayerFactors) nc.C_out[o] = clip_factor(norm_of(sq), nc.mode, nc.R[l], nc.stability);
}

// End of every workgroup of a kernel that stores final norms, all of them from its first wave: kGroupFactors.  The norms
// are stored past the caches that another workgroup does not share and are complete before the count, whose
// last reader adds them up, nc.width lanes to a sample (all samples at one time, a lane up to eight of them), in the order
// of the clip kernel: the same bits.  (With fences in their place, which write back and drop the whole cache, it took 1 to 2 us longer.)  lds: a
// word of the workgroup's LDS.
template <int THREADS>
__device__ __forceinline__ void finish_norms(const GroupArgs& ga, const NormClip& nc, const float* sqnorm, unsigned* lds) {
  static_assert(8 * THREADS >= kFinishLanes, "all samples at one time");
  if (nc.kind != kGroupFactors) return;
  __syncthreads();                                     // nobody reads that word any more
  if (threadIdx.x < 64) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0)
      *lds = __hip_atomic_fetch_add(nc.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (*lds != nc.blocks - 1) return;
  const int width = nc.width, sub = threadIdx.x & (width - 1), i0 = threadIdx.x / width, stride = THREADS / width;
  auto add_up = [&](auto n) {                          // samples i0, i0 + stride, ..., n of them in flight
    constexpr int N = decltype(n)::value;
    float total[N] = {};
    for (int l = sub; l < nc.L; l += 64) {             // more than once for 64 lanes only
      float v[N];
#pragma unroll
      for (int q = 0; q < N; ++q) {
        const int i = i0 + q * stride;
        v[q] = i < ga.B ? __hip_atomic_load(&sqnorm[(size_t)l * ga.B + i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.f;
      }
#pragma unroll
      for (int q = 0; q < N; ++q) total[q] += v[q];
    }
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int i = i0 + q * stride;
      if (i >= ga.B) break;                            // of all the sample's lanes
      for (int off = width / 2; off > 0; off >>= 1) total[q] += __shfl_xor(total[q], off);
      const float norm = norm_of(total[q]);
      if (sub == 0) {
        nc.C_out[i] = clip_factor(norm, nc.mode, nc.R[0], nc.stability);
        if (nc.norm_out) nc.norm_out[i] = norm;
      }
    }
  };
  if (ga.B <= stride)
    add_up(std::integral_constant<int, 1>{});
  else
    add_up(std::integral_constant<int, 8>{});
  if (threadIdx.x == 0) *nc.counter = 0;
}

}  // namespace dpbk
