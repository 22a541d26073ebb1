// Tile sizes, input addressing and the shortcut's arithmetic of the one-launch bottleneck blocks (conv_block.hip).  Plain C++,
// compiled for the device and by host tests.
#pragma once
#include <stdint.h>

namespace hawq {

constexpr int BLOCK_TW = 14, BLOCK_TH = 8;                             // output pixels of a tile
constexpr int BLOCK_HW = 16, BLOCK_HROWS = BLOCK_TH + 2;               // its input with a border of one pixel: columns, rows

// Byte offset of image n's row y (inside the image or not) as a load's scalar offset.  Rows outside the image are read at a lane
// offset that is out of range, and the scalar offset stays inside the tensor all the same: the range check subtracts it from the
// buffer's size, and what it does with a negative difference is documented nowhere.  (The same test as the lane offset's: one
// select; clamping the row cost two scalar instructions a load and 0.1 to 0.2 % of a ResNet50 forward.)
constexpr int32_t block_input_row(int n, int y, int H, int W, int pixel_bytes) {
    return (unsigned)y < (unsigned)H ? (n * H + y) * W * pixel_bytes : 0;
}

// The shortcut of an unsigned byte in floating point, exactly:  (r*rb + 2^(rc-1)) >> rc  is the integer nearest to
// x = r*rb / 2^rc, a half rounded up.  With the multiplier raised to (256 rb + 1) / 2^(rc+8) the product is x + r / 2^(rc+8):
// nothing that is a multiple of 2^-rc lies between the two (r < 256), a half is no tie any more, and one fused multiply-add with
// 1.5 * 2^23 rounds to the nearest integer -- the result's bits are kResMagic + the term.  24 bits hold 256 rb + 1 for rb < 2^16,
// and rc >= 2 keeps the term below 2^22.
constexpr int32_t kResMagic = 0x4B400000;
constexpr float kResMagicF = 12582912.f;               // 1.5 * 2^23, whose bits are kResMagic
constexpr bool res_float_ok(int32_t rb, int32_t rc) { return rb < 65536 && rc >= 2; }
inline int32_t res_float(int32_t rb, int32_t rc) {
    return __builtin_bit_cast(int32_t, __builtin_ldexpf((float)(256 * rb + 1), -(rc + 8)));
}
template <typename Float>                              // (a template: a plain constexpr function would have to have constant results)
constexpr int32_t res_scaled(Float r, int32_t rf) {
    return __builtin_bit_cast(int32_t, __builtin_fmaf(r, __builtin_bit_cast(float, rf), kResMagicF));
}

}  // namespace hawq
