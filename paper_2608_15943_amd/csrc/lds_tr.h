// LDS tiles read along their rows with the gfx950 transpose read (ds_read_b64_tr_b16),
// for the backward attention kernels.
#pragma once

#include "common.h"

namespace kvp {

// Staged tiles use a sub-tiled LDS layout: an NR x NC bf16 tile is stored as NC / 32 blocks
// of 32 columns, each NR rows of 64 bytes; 16-byte chunk k (0..3) of row r of a block sits
// at position k ^ ((r >> 2) & 3).  A column-block or 16-row offset is then a constant byte
// offset (so every read below is one lane register plus an immediate), and 16 consecutive
// rows of one chunk column cover all 64 banks.
template <int NR>
__device__ __forceinline__ int sub_off(int r, int c) {
    return (c >> 5) * (NR * 64) + r * 64 + ((((c >> 3) & 3) ^ ((r >> 2) & 3)) << 4) + ((c & 7) << 1);
}

// One 1 KB direct load (16 bytes per lane) of rows 16 q .. 16 q + 15 of column block sb:
// lane i fetches the global chunk that belongs at position i % 4 of row 16 q + i / 4.
// Returns the chunk index (0..3) within the block; the caller supplies the global row.
__device__ __forceinline__ int sub_chunk(int lane) { return (lane & 3) ^ ((lane >> 4) & 3); }

// The kernels read two kinds of fragments, their lane addresses computed once (asm reads with
// immediate offsets for row blocks, column blocks and stages):
//   row fragment: columns c .. c + 7 (c % 8 == 0) of row r, one 16-byte read at sub_off(r, c);
//   transposed fragment (r0, c0): lane (n = lane % 32, hi = lane / 32) receives
//     tile[r0 + 8 hi + j][c0 + n], j = 0 .. 7 (r0 % 16 == 0, c0 % 32 == 0), by two
//     ds_read_b64_tr_b16: in each group G of 16 lanes, lane 4 a + e receives element e of the 8
//     bytes addressed by lanes a, a + 4, a + 8, a + 12 of the group, so lane i of a group
//     addresses row r0 + 8 (G / 2) + i / 4 (+ 4 for the second read) at column
//     c0 + 16 (G % 2) + 4 (i % 4); permuted (bits 2 and 3 of n swapped), i % 4 has its two
//     bits swapped.

}  // namespace kvp
