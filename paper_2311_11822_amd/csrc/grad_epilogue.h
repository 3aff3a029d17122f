// Epilogue shared by the matrix-core gradient kernels: weighted sum -> old value when accumulating ->
// noise -> store, in fp32 or in the operands' 16-bit storage type.
#pragma once

#include <type_traits>

#include "dp_internal.h"

namespace dpbk {

typedef __attribute__((ext_vector_type(4))) float f32x4v;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4v;
typedef __attribute__((address_space(3))) f32x4v lds_f4;

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

// The kernel's copy of what the noise needs, read once from the kernel arguments into registers.
struct TileNoise {
  float stddev;
  uint32_t step_lo, step_hi;
  uint64_t lo, hi, layer_off;
  RoundKeys rk;
};

__device__ __forceinline__ TileNoise load_tile_noise(const NoiseArgs& args, int layer) {
  int zero = 0;
  asm volatile("" : "+s"(zero));                         // where tiles come in a loop: read for each, not held beside the contraction
  const NoiseArgs& na = (&args)[zero];
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

// Output of one wave: NY 32 x 32 tiles side by side, 32 rows of 32 NY columns.
//
// The MFMAs take the g fragment as first operand and the a fragment as second, so a wave holds the transposed product:
// lane l has row (l & 31) of a tile and the columns 8 q + 4 (l >> 5) + e (q, e = 0 .. 3) in register 4 q + e.  Stored from
// there, an instruction touches 32 rows, 32 bytes of each (16-bit output: 16), and L2 takes four (eight) requests for a line:
// that many requests, not the bytes, were the bound of short contractions (104 M elements of fp32: 13 M requests of 32
// bytes, 3.3 M lines).  So the values go through LDS, a region of the wave's own, and every store instruction writes whole
// rows of the wave's piece, 16 bytes a lane.  Steps, us, from the registers and through LDS: 2 x 32 tokens, 44 layers of width
// 1344 stored in 16 bits 290, 255; 2 x 32, 44 of width 1488 in fp32 355, 312; 18 tokens of 3 samples, 48 of width 320 40, 34;
// 4096 tokens, 144 of width 1280 7.31, 7.36 ms.
//
// Whole rows leave by streaming (nontemporal) stores where the caller says so (rows_stream in dp_api.hip): cached stores of what the
// launch does not read only push the operands out of the caches.  Gradients with noise, us, cached and streaming: 24 layers 1280 x 1280,
// 16 x 112 tokens 186, 169; 32 x 48 182, 170; 24 GPT layers of width 1024 (fp16), 10 x 100 241, 221; 48 of width 1280, 8 x 512 1845,
// 1840.  (Of the registers' 32-byte pieces they took four times as long.)
template <int NY>
struct WavePiece {
  static constexpr int H = 32, W = 32 * NY;            // rows, columns
  static constexpr int STRIDE = 4 * W + 16;            // bytes of a row: 16 of them begin in different banks
  static constexpr int BYTES = H * STRIDE;
  const f32x16* acc;                                   // its tiles' sums, first row and column
  int row0, col0;
  __device__ __forceinline__ void put(unsigned lds, int lane) const {
#pragma unroll
    for (int y = 0; y < NY; ++y)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *(lds_f4*)(uintptr_t)(lds + (lane & 31) * STRIDE + (32 * y + 8 * q + 4 * (lane >> 5)) * 4) =
            f32x4v{acc[y][4 * q], acc[y][4 * q + 1], acc[y][4 * q + 2], acc[y][4 * q + 3]};
  }
  // Columns 4 quad .. 4 quad + 3 of a row
  static __device__ __forceinline__ unsigned at(unsigned lds, int row, int quad) { return lds + row * STRIDE + quad * 16; }
};

// H rows of 2 NY tiles of 16 x 16: lane l has row l & 15 and the columns 4 (l >> 4) + e of a tile in register e; the tiles 16 rows
// down are PITCH further on.  Without room between the rows: 16 bytes are where the row's number exclusive-or'd says, so
// that 16 rows' are in different banks.
template <int NY, int H_, int PITCH>
struct WavePiece16 {
  static constexpr int H = H_, W = 32 * NY;
  static constexpr int BYTES = H * W * 4;
  const f32x4v* acc;
  int row0, col0;
  __device__ __forceinline__ void put(unsigned lds, int lane) const {
#pragma unroll
    for (int x = 0; x < H / 16; ++x)
#pragma unroll
      for (int y = 0; y < 2 * NY; ++y)
        *(lds_f4*)(uintptr_t)at(lds, 16 * x + (lane & 15), 4 * y + (lane >> 4)) = acc[PITCH * x + y];
  }
  static __device__ __forceinline__ unsigned at(unsigned lds, int row, int quad) {
    return lds + row * (W * 4) + ((quad ^ (NY == 1 ? row >> 1 & 7 : row & 15)) << 4);
  }
};

// How a wave's piece leaves: N store instructions of ROWS rows, LANES lanes to a row, VEC columns a lane.
template <class Piece, bool OUT16>
struct RowStores {
  static constexpr int VEC = OUT16 ? 8 : 4, LANES = Piece::W / VEC, ROWS = 64 / LANES, N = Piece::H / ROWS;
};

// The old values of a piece, asked for before its sums go through LDS: a wave has those of 32 rows on their way, of two pieces
// where a piece is 16.  Accumulating gradients, us, one piece's and two: 2 x 82 tokens, 20 layers of GPT width 1176 169.5, 159.9; 8 x 128,
// 48 of width 768 266, 256; 3 x 577, 24 of 1840 x 1840 379, 371; on average 4 % of 128 x 128 tiles, 7 % of joined ones in 16 bits.
template <class Piece, bool OUT16>
struct OldRows {
  u32x4v raw[RowStores<Piece, OUT16>::N];
  __device__ __forceinline__ void load(const float* out32, int row0, int col0, int d, int p, int lane) {
    using S = RowStores<Piece, OUT16>;
    const int row = row0 + lane / S::LANES, col = col0 + lane % S::LANES * S::VEC;
    const char* at = reinterpret_cast<const char*>(out32) + ((size_t)row * p + col) * (OUT16 ? 2 : 4);
    const size_t step = (size_t)S::ROWS * p * (OUT16 ? 2 : 4);
#pragma unroll
    for (int n = 0; n < S::N; ++n) {
      raw[n] = u32x4v{0, 0, 0, 0};
      if (row + n * S::ROWS < d && col < p) raw[n] = *reinterpret_cast<const u32x4v*>(at + n * step);
    }
  }
};

// What the wave's lanes wrote to its region is there for its other lanes, and what they read has been read: LDS serves a
// wave in order, so this only holds the compiler to it (no instruction).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// acc * held (+ old value) (+ noise of eq. (1)) -> out, in fp32 or the operands' 16-bit type; lds: the wave's Piece::BYTES;
// ready: called before the first store.
// Noise: same values as the separate pass, which indexes the generator by global element too; requires layer_off and d_out
// to be multiples of 4, as a lane's four columns are one block of the generator.
enum Rows { kAdd, kStream, kKeep };                      // old values added; by streaming stores; through the caches
template <bool F16, bool NOISE, bool OUT16, Rows ROWS_GO, class Piece, class Ready>
__device__ __forceinline__ void store_rows(const Piece& piece, const OldRows<Piece, OUT16>& old, float held, unsigned lds, float* out32,
                                           int d, int p, const TileNoise& na, int lane, Ready ready) {
  constexpr bool ACCUMULATE = ROWS_GO == kAdd;
  const int row0 = piece.row0, col0 = piece.col0;
  piece.put(lds, lane);
  wave_lds_fence();
  bool noisy = false, whole = false;
  if constexpr (NOISE) {
    const int rows = min(Piece::H, d - row0), cols = min(Piece::W, p - col0);
    const uint64_t e_first = na.layer_off + (uint64_t)row0 * p + col0;
    const uint64_t e_last = na.layer_off + (uint64_t)(row0 + rows - 1) * p + (col0 + cols - 1);
    noisy = rows > 0 && cols > 0 && e_last >= na.lo && e_first < na.hi;              // wave-uniform
    whole = e_first >= na.lo && e_last < na.hi;
  }
  constexpr int VEC = RowStores<Piece, OUT16>::VEC, LANES = RowStores<Piece, OUT16>::LANES;
  constexpr int ROWS = RowStores<Piece, OUT16>::ROWS, N = RowStores<Piece, OUT16>::N;
  constexpr int BLOCKS = VEC / 4, U = 4 / BLOCKS;                                     // U at a time: four generator blocks
  static_assert(N % U == 0, "whole groups");
  const int row = row0 + lane / LANES, col = col0 + lane % LANES * VEC;
  const size_t at = (size_t)row * p + col, step = (size_t)ROWS * p;      // the lane's first element; from one to the next
  float v[N][VEC];
#pragma unroll
  for (int n = 0; n < N; ++n)
#pragma unroll
    for (int b = 0; b < BLOCKS; ++b) {
      const f32x4v w = *(const lds_f4*)(uintptr_t)Piece::at(lds, lane / LANES + n * ROWS, lane % LANES * BLOCKS + b);
#pragma unroll
      for (int k = 0; k < 4; ++k) v[n][4 * b + k] = ACCUMULATE ? w[k] : w[k] * held;
    }
  wave_lds_fence();                                      // the wave's next piece is written over it
#pragma unroll
  for (int n = 0; n < N; n += U) {
    if constexpr (ACCUMULATE) {
#pragma unroll
      for (int u = n; u < n + U; ++u)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if constexpr (OUT16) {
            v[u][2 * k] = fmaf(v[u][2 * k], held, from_half_bits<F16>((uint16_t)(old.raw[u][k] & 0xFFFFu)));
            v[u][2 * k + 1] = fmaf(v[u][2 * k + 1], held, from_half_bits<F16>((uint16_t)(old.raw[u][k] >> 16)));
          } else {
            v[u][k] = fmaf(v[u][k], held, __uint_as_float(old.raw[u][k]));       // one rounding
          }
        }
    }
    if (NOISE && noisy) {
      // The four blocks side by side, and all of them before the test of the shard's ends, into which the compiler would
      // move the chains one by one.  (Lanes past the layer's edge draw values that are not stored.)
      const uint64_t e = na.layer_off + at + n * step;
      uint64_t block[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) block[q] = ((e + q / BLOCKS * step) >> 2) + q % BLOCKS;
      float z[4][4];
      normal_blocks(block, na.step_lo, na.step_hi, na.rk, z);
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(z[q][k]));
      if (whole) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int k = 0; k < VEC; ++k) v[n + u][k] = fmaf(na.stddev, z[u * BLOCKS + k / 4][k % 4], v[n + u][k]);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int k = 0; k < VEC; ++k)
            if (e + u * step + k >= na.lo && e + u * step + k < na.hi)
              v[n + u][k] = fmaf(na.stddev, z[u * BLOCKS + k / 4][k % 4], v[n + u][k]);
      }
    }
    if (n == 0) ready();
    u32x4v w[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if constexpr (OUT16)
          w[u][k] = (uint32_t)to_half_bits<F16>(v[n + u][2 * k]) | ((uint32_t)to_half_bits<F16>(v[n + u][2 * k + 1]) << 16);
        else
          w[u][k] = __float_as_uint(v[n + u][k]);
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (row + (n + u) * ROWS < d && col < p) {
        u32x4v* to = reinterpret_cast<u32x4v*>(reinterpret_cast<char*>(out32) + (at + (n + u) * step) * (OUT16 ? 2 : 4));
        if constexpr (ROWS_GO == kStream)
          __builtin_nontemporal_store(w[u], to);
        else
          *to = w[u];
      }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// COUNT pieces of the wave; ready: called before the first store.  The three forms lie one behind the other: with a branch at every group of
// stores a wave fetches both forms' code (seven 1024 x 1024 layers, 4 x 256 tokens 20.6 us with one form, 20.8 so).
template <int COUNT, bool F16, bool NOISE, bool OUT16, class PieceOf, class Ready>
__device__ __forceinline__ void store_pieces(PieceOf piece, bool accumulate, bool stream, float held, unsigned lds, float* out32, int d, int p,
                                             const TileNoise& na, int lane, Ready ready) {
  using Piece = decltype(piece(0));
  // With noise in fp32 a 256 x 256 tile has no registers for two pieces', and 128 x 128 ones take 1 % more.
  constexpr int AHEAD = COUNT % 2 == 0 && Piece::H == 16 && (OUT16 || !NOISE) ? 2 : 1;
  auto store_all = [&](auto rows) {
    constexpr Rows GO = decltype(rows)::value;
#pragma unroll
    for (int i = 0; i < COUNT; i += AHEAD) {
      OldRows<Piece, OUT16> old[AHEAD];
#pragma unroll
      for (int j = 0; j < AHEAD; ++j)
        if (GO == kAdd) old[j].load(out32, piece(i + j).row0, piece(i + j).col0, d, p, lane);
#pragma unroll
      for (int j = 0; j < AHEAD; ++j)
        store_rows<F16, NOISE, OUT16, GO>(piece(i + j), old[j], held, lds, out32, d, p, na, lane, [&]() {
          if (i + j == 0) ready();
        });
    }
  };
  if (accumulate) {
    store_all(std::integral_constant<Rows, kAdd>{});
  } else if (stream) {
    store_all(std::integral_constant<Rows, kStream>{});
    asm volatile("");                                    // or these two become one, through the caches
  } else {
    store_all(std::integral_constant<Rows, kKeep>{});
  }
}

}  // namespace dpbk
