// Row tiles on their way global memory -> LDS -> matrix operands, for tiles that are 128, 64 or 32 columns wide
// (grad_packed.hip, perex_narrow.hip): k-blocks of 32 rows, four waves, no register staging.
#pragma once

#include "dp_internal.h"
#include "lds_dma.h"

namespace dpbk {

// Loads of one operand per wave and k-block.
template <int W>
constexpr int kRowLoads = W == 128 ? 2 : 1;

// K: rows of a matrix instruction, 16 (32x32x16: 32 columns) or 32 (16x16x32: 16 columns).
//
// The lanes' 16-byte chunk c of row r holds logical chunk row_chunk(c, r): the four consecutive rows that
// one transposing read touches (64 bytes of each; K = 32: 32 bytes, and of four rows eight below) spread over the 256
// bytes of banks.
template <int W, int K>
__device__ __forceinline__ int row_chunk(int chunk, int row) {
  if (K == 32) chunk ^= (row >> 3 & 1) << 1;
  if (W == 128) return chunk ^ ((row & 3) << 2);       // 256-byte rows: each row a bank group of its own
  if (W == 64) return chunk ^ ((row & 2) << 1);        // 128-byte rows: the second pair moves by 64 bytes
  return chunk;                                        // 64-byte rows: as they lie
}

// One operand: W columns from col0 of a row-major [rows, width] matrix.  W = 128: load j of a wave covers
// rows 16 j + 4 wave + (lane >> 4); W = 64: rows 8 wave + (lane >> 3); W = 32: half the lanes cover rows
// 8 wave + (lane >> 2).
template <int W, int K>
struct RowOperand {
  i32x4 rsrc;
  unsigned v, step;                // byte offset of this lane's chunk; bytes per 16 rows
  unsigned lds;                    // first LDS byte of this wave's loads inside a stage
  __device__ __forceinline__ void init(const void* base, int64_t rows, int width, int col0, unsigned lds_base, int wave,
                                       int lane) {
    constexpr int CHUNKS = W / 8;
    rsrc = make_rsrc(base, (unsigned)(rows * width * 2));
    const int row = wave * (W == 128 ? 4 : 8) + (lane / CHUNKS) % (W == 32 ? 8 : 64);
    const int chunk = row_chunk<W, K>(lane % CHUNKS, row);
    v = col0 + chunk * 8 < width ? (unsigned)(row * width + col0 + chunk * 8) * 2u : OOB;
    step = 32u * width;
    lds = lds_base + wave * (W == 32 ? 512 : 1024);
  }
  __device__ __forceinline__ void issue(unsigned stage_off, int lane) {
    if (W == 128) {
      load_to_lds(rsrc, v, 0, lds + stage_off);
      load_to_lds(rsrc, v + step, 0, lds + stage_off + 4096);
    } else if (W == 64 || lane < 32) {
      load_to_lds(rsrc, v, 0, lds + stage_off);
    }
    v += 2 * step;                 // rows past the last one lie past the descriptor's size: zeros
  }
};

// LDS byte of a lane's first transposing read of the 32-column (K = 32: 16-column) tile at col0, with b = lane >> 4,
// s = lane & 15: k row 8 (b >> 1) + (s >> 2), columns 16 (b & 1) + 4 (s & 3) (K = 32: 8 b + (s >> 2), 4 (s & 3)).
template <int W, int K>
__device__ __forceinline__ unsigned row_frag_base(int col0, int lane) {
  const int b = lane >> 4, s = lane & 15;
  const int row = 8 * (K == 32 ? b : b >> 1) + (s >> 2), col = col0 + (K == 32 ? 0 : 16 * (b & 1)) + 4 * (s & 3);
  return row * (W * 2) + (row_chunk<W, K>(col >> 3, row) << 4) + (s & 1) * 8;
}
template <int W>
__device__ __forceinline__ bf16x8 read_row_frag(unsigned addr) {
  Frag f;
  f.h[0] = lds_read_tr(addr);
  f.h[1] = lds_read_tr(addr + 4 * W * 2);
  return f.v;
}

}  // namespace dpbk
