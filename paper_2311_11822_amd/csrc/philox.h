// Counter-based Gaussian generator shared by the noise pass and by the gradient kernels that
// add the noise in their epilogue: Philox4x32-10 (Salmon et al., SC'11) + Box-Muller.
// Block k of the element stream (elements 4k .. 4k+3) has counter (k_lo, k_hi, step_lo,
// step_hi) and key (seed_lo, seed_hi); u = ((x >> 9) + 1/2) 2^-23;
// (z_4k, z_4k+1) = sqrt(-2 ln u(x0)) (cos, sin)(2 pi u(x1)), (z_4k+2, z_4k+3) likewise from
// (x2, x3).  log2 / sin / cos use the hardware units (sin and cos take their argument in
// revolutions, which is exactly the uniform variate; measured absolute error 1.3e-7, log2
// relative 1.2e-7).
// Bound by the vector ALU, and by itself by the latency of its chain: blocks that a thread needs together go through the
// rounds side by side.  Two waves per SIMD with four blocks in flight: 368 G blocks/s with the compiler's two-input
// exclusive ors and a conversion to float for the uniform variate, 460 with three-input ones, 487 as it is.  In the
// gradient kernels' epilogue with four blocks side by side too: 20 x 32 tokens, 32 layers of width 808, 249 -> 225 us; 6 x 32,
// 20 layers of width 896, 122 -> 104 us (9 of these with the chains one after the other).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dpbk {

constexpr uint32_t kMulA = 0xD2511F53u;
constexpr uint32_t kMulB = 0xCD9E8D57u;
constexpr uint32_t kWeylA = 0x9E3779B9u;
constexpr uint32_t kWeylB = 0xBB67AE85u;

struct RoundKeys {
  uint32_t k[10][2];
};

inline RoundKeys make_round_keys(uint64_t seed) {
  RoundKeys rk;
  uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
  for (int r = 0; r < 10; ++r) {
    rk.k[r][0] = k0;
    rk.k[r][1] = k1;
    k0 += kWeylA;
    k1 += kWeylB;
  }
  return rk;
}

// a ^ b ^ c in one instruction (the compiler makes two of them).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// N blocks, one after the other inside each round: a block by itself is a chain of some thirty dependent instructions.
template <int N>
__device__ __forceinline__ void philox_blocks(const uint64_t (&block)[N], uint32_t step_lo, uint32_t step_hi,
                                              const RoundKeys& rk, uint32_t (&x)[N][4]) {
#pragma unroll
  for (int n = 0; n < N; ++n) {
    x[n][0] = (uint32_t)block[n];
    x[n][1] = (uint32_t)(block[n] >> 32);
    x[n][2] = step_lo;
    x[n][3] = step_hi;
  }
#pragma unroll
  for (int r = 0; r < 10; ++r)
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const uint64_t pa = (uint64_t)kMulA * x[n][0], pb = (uint64_t)kMulB * x[n][2];
      x[n][0] = xor3((uint32_t)(pb >> 32), x[n][1], rk.k[r][0]);
      x[n][2] = xor3((uint32_t)(pa >> 32), x[n][3], rk.k[r][1]);
      x[n][1] = (uint32_t)pb;
      x[n][3] = (uint32_t)pa;
    }
}

__device__ __forceinline__ void philox_block(uint64_t block, uint32_t step_lo, uint32_t step_hi,
                                             const RoundKeys& rk, uint32_t x[4]) {
  const uint64_t blocks[1] = {block};
  uint32_t y[1][4];
  philox_blocks(blocks, step_lo, step_hi, rk, y);
#pragma unroll
  for (int k = 0; k < 4; ++k) x[k] = y[0][k];
}

// u = ((x >> 9) + 1/2) 2^-23: x >> 9 as the mantissa of a number in [1, 2), less 1 - 2^-24; exact in fp32.
__device__ __forceinline__ float to_uniform(uint32_t x) {
  return __uint_as_float(__builtin_amdgcn_alignbit(0x7Fu, x, 9)) - 0x1.fffffep-1f;
}

__device__ __forceinline__ void box_muller(uint32_t xa, uint32_t xb, float& z0, float& z1) {
  const float ua = to_uniform(xa), ub = to_uniform(xb);
  // -2 ln u = (-2 ln 2) log2 u
  const float r = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(ua));
  z0 = r * __builtin_amdgcn_cosf(ub);
  z1 = r * __builtin_amdgcn_sinf(ub);
}

// The four normals of one block.
__device__ __forceinline__ void normal_block(uint64_t block, uint32_t step_lo, uint32_t step_hi,
                                             const RoundKeys& rk, float z[4]) {
  uint32_t x[4];
  philox_block(block, step_lo, step_hi, rk, x);
  box_muller(x[0], x[1], z[0], z[1]);
  box_muller(x[2], x[3], z[2], z[3]);
}

// Of N blocks.
template <int N>
__device__ __forceinline__ void normal_blocks(const uint64_t (&block)[N], uint32_t step_lo, uint32_t step_hi,
                                              const RoundKeys& rk, float (&z)[N][4]) {
  uint32_t x[N][4];
  philox_blocks(block, step_lo, step_hi, rk, x);
#pragma unroll
  for (int n = 0; n < N; ++n) {
    box_muller(x[n][0], x[n][1], z[n][0], z[n][1]);
    box_muller(x[n][2], x[n][3], z[n][2], z[n][3]);
  }
}

}  // namespace dpbk
