// Tile sizes and input addressing of the one-launch bottleneck blocks (conv_block.hip).  Plain C++, compiled for the device and by a
// host test.
#pragma once
#include <stdint.h>

namespace hawq {

constexpr int BLOCK_TW = 14, BLOCK_TH = 8;                             // output pixels of a tile
constexpr int BLOCK_HW = 16, BLOCK_HROWS = BLOCK_TH + 2;               // its input with a border of one pixel: columns, rows

// Byte offset of image n's row y (inside the image or not) as a load's scalar offset.  Rows outside the image are read at a lane
// offset that is out of range, and the scalar offset stays inside the tensor all the same: the range check subtracts it from the
// buffer's size, and what it does with a negative difference is documented nowhere.
constexpr int32_t block_input_row(int n, int y, int H, int W, int pixel_bytes) {
    const int inside = y < 0 ? 0 : y < H ? y : H - 1;
    return (n * H + inside) * W * pixel_bytes;
}

}  // namespace hawq
