// Where the output tiles of the 6-bit float GEMM kernel lie and how their rows are stored.  Plain C++, used on both sides.
#pragma once

#include <stdint.h>

namespace sq {

// First row (column) of tile number `index` of `size` rows: the last tile ends with the matrix and overlaps its neighbour.
constexpr int fp6_tile_origin(int index, int size, int extent)
{
    return index * size < extent - size ? index * size : extent - size;
}

// What the host knows: 16-byte stores are possible where a tile's first channel is a multiple of eight.
constexpr bool fp6_rows_aligned(uintptr_t y, int64_t ldy) { return y % 16 == 0 && ldy % 8 == 0; }

// ... and a tile takes them if it begins there: all do but, where N is no multiple of eight, the last of a row of tiles.
constexpr bool fp6_vector_stores(bool rows_aligned, int col0) { return rows_aligned && col0 % 8 == 0; }

}  // namespace sq
