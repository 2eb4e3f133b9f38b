// pieces.h -- which 16 bytes of an operand each piece of gemm_tile_kernel's stages reads
// (kern_tile.h says why these stay inside the operand).  Host and device.
#pragma once

#include <stdint.h>

namespace gemm {

// K-contiguous rows (A, column-major B): byte offset of chunk c of tile row `row`, from the
// tile's first row at the stage's start.  Rows past `last`, the tile's last valid one, repeat it.
constexpr int64_t row_piece(int row, int last, int64_t ld_bytes, int c) {
    return int64_t(row < last ? row : last) * ld_bytes + c * 16;
}

// ... and in the stage that ends K after rem_bytes: how far back of that offset the piece is
// read, to end at the row's end, and shifted down by afterwards.
constexpr int row_piece_back(int c, int rem_bytes) {
    const int over = c * 16 + 16 - rem_bytes;
    return over > 0 ? over : 0;
}

// Row-major B: the column that the piece for columns from `col` starts at.  Pieces wholly past N
// take the last column on.
constexpr int64_t col_piece(int64_t col, int64_t N) { return col < N ? col : N - 1; }

// ... and in the stage that ends K: ending at the row's end, in one of the `rem` rows left.
constexpr int64_t col_piece_tail(int64_t col, int64_t N, int elems) { return col + elems <= N ? col : N - elems; }
constexpr int row_tail(int row, int rem) { return row < rem ? row : rem - 1; }

}  // namespace gemm
