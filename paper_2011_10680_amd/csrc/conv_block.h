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

// The shortcut of an unsigned byte in floating point, exactly:  (r*rb + 2^(rc-1)) >> rc  is the integer nearest to
// x = r*rb / 2^rc, a half rounded up.  With the multiplier raised to (256 rb + 1) / 2^(rc+8) the product is x + r / 2^(rc+8):
// nothing that is a multiple of 2^-rc lies between the two (r < 256), a half is no tie any more, and one fused multiply-add with
// 1.5 * 2^23 rounds to the nearest integer -- the result's bits are kResMagic + the term.  24 bits hold 256 rb + 1 for rb < 2^16,
// and rc >= 2 keeps the term below 2^22.
constexpr int32_t kResMagic = 0x4B400000;
inline bool res_float_ok(int32_t rb, int32_t rc) { return rb < 65536 && rc >= 2; }
inline int32_t res_float(int32_t rb, int32_t rc) {
    return __builtin_bit_cast(int32_t, __builtin_ldexpf((float)(256 * rb + 1), -(rc + 8)));
}

hawq_status launch_block64(const BlockArgs &a, hipStream_t s);

}  // namespace hawq
