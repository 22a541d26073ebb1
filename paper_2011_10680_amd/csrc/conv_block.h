// A bottleneck block at 64 channels as one launch (conv_block.hip).
#pragma once
#include "common.h"
#include "conv_block_plan.h"

namespace hawq {

struct BlockArgs {
    const uint8_t *x;            // [N][H][W][256] unsigned bytes up to 127, or packed 4-bit (x4); with w4 [N][H][W][64] bytes
    uint8_t *y;                  // [N][H][W][256] bytes or packed 4-bit (y4)
    int32_t N, H, W;
    const uint8_t *w1, *w2, *w3, *w4;   // weights in fragment order (bytes; w1 of a packed input in that input's order); w4: the
                                        // convolution on the shortcut, or null
    const int32_t *par;          // [9 arrays]: bias and b << (32 - c) of the 1x1 (64 each) and of the 3x3 (64), of the closing 1x1 (256),
                                 // the shortcut's multiplier << (t - its shift) (256), bias and b << (32 - c) of w4's convolution (256)
    int32_t hi1, hi2, lo3, hi3;  // clamps (the first two from 0)
    int32_t t, mid8;             // shift of the shortcut's multipliers; w4: its result passes through a signed byte first
    int32_t x4, y4;
    int32_t flt;                 // without w4, bytes: the shortcut's multipliers are floats (res_float), t is not looked at
    int32_t tiles_x, tiles_y, n_tiles;  // set by the launcher
};
constexpr int BLOCK64_PAR = 1536;       // words of par

hawq_status launch_block64(const BlockArgs &a, hipStream_t s);

}  // namespace hawq
