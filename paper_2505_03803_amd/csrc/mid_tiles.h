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

// Weights unrounded, M rows of x: 16 MF rows of x in a workgroup, evenly over the fewest workgroups of at most 64; 16 NF rows of W, where
// `narrow` workgroups of 32 hold the launch: up to one per compute unit 32 win, up to half of that 16 (see midbatch.hip).
constexpr int mid_exact_mf(int M) { return ((M + (M + 63) / 64 - 1) / ((M + 63) / 64) + 15) / 16; }
constexpr int mid_exact_nf(int mf, long long narrow) { return narrow <= 128 ? 1 : narrow <= 256 || mf == 1 ? 2 : 4; }
// The instances that there are.
constexpr bool mid_exact_instance(int mf, int nf) { return mf >= 1 && mf <= 4 && (nf == 1 || nf == 2 || (nf == 4 && mf > 1)); }

}  // namespace rwkvq
