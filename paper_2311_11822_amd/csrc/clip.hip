// Cross-layer norm accumulation and clip factors (section 2.1 of the paper; all-layer
// clipping = one group, eq. (1) with M = 1).  A few hundred floats: one tiny launch.
#include "clip.h"
#include "norm_partials.h"

namespace dpbk {

namespace {

__global__ void __launch_bounds__(64)
clip_factor_kernel(const float* __restrict__ sqnorm, int L, int B, int mode, float R,
                   float stability, float* __restrict__ C_out, float* __restrict__ norm_out) {
  const int i = blockIdx.x;                                  // one wave per sample
  const float total = column_sum(sqnorm, B, i, 0, L, threadIdx.x);
  if (threadIdx.x != 0) return;
  const float norm = norm_of(total);
  C_out[i] = clip_factor(norm, mode, R, stability);
  if (norm_out) norm_out[i] = norm;
}

// The last norm launch's partial sums and the clip factors in one launch: both are chains of launch and memory latencies.
// One workgroup to a sample; `width` lanes add the partial sums of a layer each, as many layers at a time as that
// gives, then the first wave adds the layers, in the order of the two kernels: the same bits.  Nine samples of
// ten layers 72 wide: a step 32.9 -> 30.2 us; two samples of 768-wide layers 67.0 -> 66.2.
constexpr int kClipThreads = 1024, kClipLayers = (kMaxGroup + kClipThreads / 64 - 1) / (kClipThreads / 64);
__global__ void __launch_bounds__(kClipThreads)
norm_clip_kernel(const GroupArgs ga, const float* __restrict__ partials, float* __restrict__ sqnorm, int L, int width,
                 int mode, float R, float stability, float* __restrict__ C_out, float* __restrict__ norm_out) {
  extern __shared__ float rows[];                            // [L]
  const int i = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = threadIdx.x & (width - 1), groups = kClipThreads / width, group = threadIdx.x / width;
  float sum[kClipLayers];
#pragma unroll
  for (int q = 0; q < kClipLayers; ++q) {
    const int j = group + q * groups;
    sum[q] = j < ga.n_layers ? partial_sum(ga.layer[j], i, partials, sub, width) : 0.f;
  }
  if (ga.n_layers < L) {
    for (int l = threadIdx.x; l < L; l += kClipThreads) rows[l] = sqnorm[(size_t)l * ga.B + i];
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < kClipLayers; ++q) {
    const int j = group + q * groups;
    if (j < ga.n_layers && sub == 0) {                       // the row as read was not this call's
      rows[ga.layer[j].sq_index] = sum[q];
      sqnorm[(size_t)ga.layer[j].sq_index * ga.B + i] = sum[q];
    }
  }
  __syncthreads();
  if (wave != 0) return;
  float total = 0.f;
  for (int l = lane; l < L; l += 64) total += rows[l];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) total += __shfl_xor(total, off);
  if (lane != 0) return;
  const float norm = norm_of(total);
  C_out[i] = clip_factor(norm, mode, R, stability);
  if (norm_out) norm_out[i] = norm;
}

// Group-wise clipping (eq. (1) with M groups): group m owns the rows
// [begin[m], begin[m+1]) of sqnorm and has threshold R[m].  Up to kGroupsPerLaunch groups
// travel in the kernel arguments.
constexpr int kGroupsPerLaunch = 256;
struct GroupedClipArgs {
  int n_groups;
  int first_group;
  int begin[kGroupsPerLaunch + 1];
  float R[kGroupsPerLaunch];
};

__global__ void __launch_bounds__(64)
clip_factor_grouped_kernel(const float* __restrict__ sqnorm, int B, int mode, float stability,
                           float* __restrict__ C_out, float* __restrict__ norm_out,
                           const GroupedClipArgs ga) {
  const int i = blockIdx.x, m = blockIdx.y;                  // one wave per (sample, group)
  const float total = column_sum(sqnorm, B, i, ga.begin[m], ga.begin[m + 1], threadIdx.x);
  if (threadIdx.x != 0) return;
  const float norm = norm_of(total);
  const float c = clip_factor(norm, mode, ga.R[m], stability);
  const size_t o = (size_t)(ga.first_group + m) * B + i;
  C_out[o] = c;
  if (norm_out) norm_out[o] = norm;
}

}  // namespace

dp_status launch_clip_factors_grouped(const float* sqnorm, int B, const int32_t* group_begin, int M,
                                      const float* R, int mode, float stability, float* C_out,
                                      float* norm_out, hipStream_t s) {
  for (int first = 0; first < M; first += kGroupsPerLaunch) {
    GroupedClipArgs ga;
    ga.n_groups = M - first < kGroupsPerLaunch ? M - first : kGroupsPerLaunch;
    ga.first_group = first;
    for (int m = 0; m <= ga.n_groups; ++m) ga.begin[m] = group_begin[first + m];
    for (int m = 0; m < ga.n_groups; ++m) ga.R[m] = R[first + m];
    hipLaunchKernelGGL(clip_factor_grouped_kernel, dim3(B, ga.n_groups), dim3(64), 0, s,
                       sqnorm, B, mode, stability, C_out, norm_out, ga);
    if (hipGetLastError() != hipSuccess) return DP_ERR_HIP;
  }
  return DP_OK;
}

bool norm_clip_supports(int L) { return L <= 8192; }

dp_status launch_norm_clip(const GroupArgs& ga, const float* partials, float* sqnorm, int L, int mode, float R,
                           float stability, float* C_out, float* norm_out, hipStream_t s) {
  int width = 1;
  for (int j = 0; j < ga.n_layers; ++j)
    while (width < 64 && width < ga.layer[j].tiles_per_sample) width *= 2;
  hipLaunchKernelGGL(norm_clip_kernel, dim3(ga.B), dim3(kClipThreads), (size_t)L * sizeof(float), s, ga, partials,
                     sqnorm, L, width, mode, R, stability, C_out, norm_out);
  return hip_status(hipGetLastError());
}

dp_status launch_clip_factors(const float* sqnorm, int L, int B, int mode, float R, float stability,
                              float* C_out, float* norm_out, hipStream_t s) {
  hipLaunchKernelGGL(clip_factor_kernel, dim3(B), dim3(64), 0, s, sqnorm, L, B, mode,
                     R, stability, C_out, norm_out);
  return hip_status(hipGetLastError());
}

}  // namespace dpbk
