// W4A4 GEMM tile kernel on the 6-bit float matrix instruction (sq_w4a4_fp6.hip).
#pragma once

#include "sq_common.h"

namespace sq {

// Shapes the kernel takes: whole K tiles and at least three of them; 225 K < 2^24, so that the fp32 accumulator holds
// every sum exactly; at least one output tile (256 x 256 or 128 x 256).
inline bool w4a4_fp6_takes(bool large, int T, int K, int N)
{
    return K % 256 == 0 && K >= 768 && K <= 65536 && T >= (large ? 256 : 128) && N >= 256;
}

// launch shapes of the kernel: 256 x 256 or 128 x 256 output tiles, four waves
sq_status launch_w4a4_fp6(bool large, const uint8_t *Qx, const float *sx, int T, int K, const uint8_t *Qw,
                          const float *sw, int N, __half *Y, int64_t ldy, int32_t *acc_dbg, hipStream_t st);

}  // namespace sq
