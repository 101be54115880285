// Where the kernels of midbatch.hip find the packed words of a wavefront's row tiles.  Plain constant expressions, which the
// kernels and host code both evaluate.
#pragma once

namespace rwkvq {

// Of the NF row tiles (16 rows of W) that a wavefront starting at row tile R0 has places for, those that a matrix of N rows (a
// multiple of 16) has, and the one that its i-th place reads: past the end the last one again.
constexpr int mid_row_tiles(int N, int R0, int NF) { return (N >> 4) - R0 < NF ? (N >> 4) - R0 : NF; }
constexpr int mid_row_tile(int i, int tiles) { return i < tiles ? i : tiles - 1; }
// Byte offset of column tile T (of KT) of a row tile, each of tile_bytes, from the wavefront's first.
constexpr int mid_tile_offset(int row_tile, int T, int KT, int tile_bytes) { return (row_tile * KT + T) * tile_bytes; }

}  // namespace rwkvq
