// Epilogue shared by the matrix-core gradient kernels: weighted sum -> old value when accumulating ->
// noise -> store, in fp32 or in the operands' 16-bit storage type.
#pragma once

#include "dp_internal.h"

namespace dpbk {

typedef __attribute__((ext_vector_type(4))) float f32x4v;

// 16-bit gradient output (mixed-precision training keeps gradients in the storage type of the
// activations: section 2.3 of the paper): the fp32 value - weighted sum, old value when
// accumulating, noise - is rounded once, to nearest even, to bf16 or IEEE binary16.
template <bool F16>
__device__ __forceinline__ uint16_t to_half_bits(float x) {
  if constexpr (F16) {
    return __builtin_bit_cast(uint16_t, (_Float16)x);
  } else {
    const uint32_t u = __float_as_uint(x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0;                    // NaN stays NaN
    return (uint16_t)((u + 0x7FFFu + ((u >> 16) & 1u)) >> 16);
  }
}
template <bool F16>
__device__ __forceinline__ float from_half_bits(uint16_t h) {
  if constexpr (F16)
    return (float)__builtin_bit_cast(_Float16, h);
  else
    return __uint_as_float((uint32_t)h << 16);
}

// Four consecutive outputs of one row: (+)= and store, fp32 (16 bytes) or 16-bit (8 bytes).
template <bool F16, bool OUT16, bool ACCUMULATE>
__device__ __forceinline__ void load_old4(const float* out32, size_t index, float (&old)[4]) {
  if constexpr (!ACCUMULATE) {
    old[0] = old[1] = old[2] = old[3] = 0.f;
  } else if constexpr (OUT16) {
    const uint2 w = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(out32) + index);
    old[0] = from_half_bits<F16>((uint16_t)(w.x & 0xFFFFu));
    old[1] = from_half_bits<F16>((uint16_t)(w.x >> 16));
    old[2] = from_half_bits<F16>((uint16_t)(w.y & 0xFFFFu));
    old[3] = from_half_bits<F16>((uint16_t)(w.y >> 16));
  } else {
    const f32x4v w = *reinterpret_cast<const f32x4v*>(out32 + index);
    old[0] = w[0]; old[1] = w[1]; old[2] = w[2]; old[3] = w[3];
  }
}
template <bool F16, bool OUT16>
__device__ __forceinline__ void store4(float* out32, size_t index, const float* v) {
  if constexpr (OUT16) {
    uint2 w;
    w.x = (uint32_t)to_half_bits<F16>(v[0]) | ((uint32_t)to_half_bits<F16>(v[1]) << 16);
    w.y = (uint32_t)to_half_bits<F16>(v[2]) | ((uint32_t)to_half_bits<F16>(v[3]) << 16);
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out32) + index) = w;
  } else {
    const f32x4v w = {v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4v*>(out32 + index) = w;
  }
}

// The kernel's copy of what tile_noise needs, read once from the kernel arguments into registers.
struct TileNoise {
  float stddev;
  uint32_t step_lo, step_hi;
  uint64_t lo, hi, layer_off;
  RoundKeys rk;
};

__device__ __forceinline__ TileNoise load_tile_noise(const NoiseArgs& na, int layer) {
  TileNoise t;
  t.stddev = na.stddev;
  t.step_lo = na.step_lo;
  t.step_hi = na.step_hi;
  t.lo = na.lo;
  t.hi = na.hi;
  t.layer_off = na.layer_off[layer];
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    t.rk.k[r][0] = na.rk.k[r][0];
    t.rk.k[r][1] = na.rk.k[r][1];
  }
  return t;
}

// Output layout.  The MFMAs take the g fragment as first operand and the a fragment as second,
// so a wave holds the transposed product: lane l has row (l & 31) of a 32 x 32 output tile and
// the columns 8 q + 4 (l >> 5) + e (q, e = 0 .. 3) in register 4 q + e: four runs of four
// consecutive columns, which are stored as 16-byte vectors (a quarter of the store
// instructions of the untransposed layout, whose lanes hold single columns) and each of which
// is exactly one block of the noise generator.
//
// Adds the noise of eq. (1) to the lane's 16 values of the tile at (tile_row0, tile_col0): same
// values as the separate noise pass, which indexes the generator by global element too.
// Requires layer_off and d_out to be multiples of 4.
__device__ __forceinline__ void tile_noise(float (&v)[16], const TileNoise& na, int tile_row0, int tile_col0,
                                           int d, int p, int lane) {
  const int rows = min(32, d - tile_row0), cols = min(32, p - tile_col0);
  if (rows <= 0 || cols <= 0) return;
  const uint64_t e_first = na.layer_off + (uint64_t)tile_row0 * p + tile_col0;
  const uint64_t e_last = na.layer_off + (uint64_t)(tile_row0 + rows - 1) * p + (tile_col0 + cols - 1);
  if (e_last < na.lo || e_first >= na.hi) return;               // wave-uniform: tile outside the shard
  const bool whole = e_first >= na.lo && e_last < na.hi;
  // The four blocks side by side, and all of them before the test of the shard's ends, into which the compiler would move
  // the chains one by one.  (Lanes past the layer's edge draw values that are not stored.)
  const uint64_t e = na.layer_off + (uint64_t)(tile_row0 + (lane & 31)) * p + (tile_col0 + 4 * (lane >> 5));
  const uint64_t block[4] = {e >> 2, (e >> 2) + 2, (e >> 2) + 4, (e >> 2) + 6};
  float z[4][4];
  normal_blocks(block, na.step_lo, na.step_hi, na.rk, z);
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(z[q][k]));
  if (whole) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) v[4 * q + k] = fmaf(na.stddev, z[q][k], v[4 * q + k]);
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint64_t at = e + 8 * q + k;
        if (at >= na.lo && at < na.hi) v[4 * q + k] = fmaf(na.stddev, z[q][k], v[4 * q + k]);
      }
  }
}

}  // namespace dpbk
