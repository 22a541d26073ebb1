// Which tiles the workgroups of a persistent kernel walk.  Plain C++, compiled for the device and by a host test.
#pragma once
#include <stdint.h>

namespace hawq {

// Tiles of workgroup b of a persistent grid of gx (a multiple of 8).  eighths: its XCD's contiguous eighth of the tiles, dealt to the
// XCD's workgroups in turn.  The kernels of a network that share this map (or xcd_remap's, which gives the same eighths) read most of
// what the kernel before them wrote from their own XCD's L2.  Measured by two plain kernels, a tensor written and read back with
// one map: 16 MB 6.6 us, 32 MB 9.7, 64 MB 21; every eighth read on another XCD than the one that wrote it: 13.9, 24.9, 31.  In the
// networks, whose kernels wait for other things as well, 1 % (ResNet50 at batch 128 1055 -> 1048 us, mixed at 256 1773 -> 1756).
// (A contiguous run per workgroup instead of turns is 2 % slower: the neighbours' walk no longer shares L2 lines.)
// Otherwise: turns over all tiles, an XCD's workgroups side by side.
struct TileWalk { int32_t first, end, step; };
constexpr TileWalk xcd_walk(uint32_t b, uint32_t gx, int32_t n_tiles, bool eighths = true) {
    const int32_t xcd = (int32_t)(b & 7), q = n_tiles >> 3, r = n_tiles & 7, own = (int32_t)(gx >> 3);
    if (!eighths) return {xcd * own + (int32_t)(b >> 3), n_tiles, (int32_t)gx};
    const int32_t lo = xcd * q + (xcd * r >> 3), hi = (xcd + 1) * q + ((xcd + 1) * r >> 3);
    return {lo + (int32_t)(b >> 3), hi, own};
}
// Eighths from 49152 output pixels on.  Below, with a round or two of tiles per workgroup, the 28 x 28 and 14 x 14 layers of ResNet50
// gain nothing and their readers lose (batch 48, 512 -> 128 at 28 x 28 behind such a layer 11.9 us, with eighths 14.1; the forward at
// batch 20 410 us, with eighths throughout 415, at 48 621 and 629; at 256, mixed widths, whose 14 x 14 layers have 50176, 1801 with
// them and 1817 with a line of 65536).
constexpr bool xcd_eighths(int64_t pixels) { return pixels >= 49152; }
// grid for it: at most `most` (a multiple of 8) workgroups, no more than the largest eighth needs
constexpr uint32_t xcd_walk_grid(int64_t n_tiles, uint32_t most) {
    const int64_t want = (n_tiles + 7) / 8 * 8;
    return want < most ? (uint32_t)want : most;
}

}  // namespace hawq
