// W4A4 GEMM tile kernel on the 6-bit float matrix instruction (sq_w4a4_fp6.hip).
#pragma once

#include "sq_common.h"

namespace sq {

// output tiles, tokens x channels; four waves each
enum class Fp6Tile { k128x192, k128x256, k256x192, k256x256 };

inline int fp6_tile_tokens(Fp6Tile tile) { return tile == Fp6Tile::k128x192 || tile == Fp6Tile::k128x256 ? 128 : 256; }
inline int fp6_tile_channels(Fp6Tile tile) { return tile == Fp6Tile::k128x192 || tile == Fp6Tile::k256x192 ? 192 : 256; }

// Shapes the kernel takes: whole K tiles and at least three of them; 225 K < 2^24, so that the fp32 accumulator holds
// every sum exactly; at least one output tile.
inline bool w4a4_fp6_takes(Fp6Tile tile, int T, int K, int N)
{
    return K % 256 == 0 && K >= 768 && K <= 65536 && T >= fp6_tile_tokens(tile) && N >= fp6_tile_channels(tile);
}

sq_status launch_w4a4_fp6(Fp6Tile tile, const uint8_t *Qx, const float *sx, int T, int K, const uint8_t *Qw,
                          const float *sw, int N, __half *Y, int64_t ldy, int32_t *acc_dbg, hipStream_t st);

}  // namespace sq
