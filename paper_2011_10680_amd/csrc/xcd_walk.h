// Which tiles the workgroups of a persistent kernel walk.  Plain C++, compiled for the device and by a host test.
#pragma once
#include <stdint.h>

namespace hawq {

// XCD-aware remap of a linear workgroup id.  Workgroups are dealt round-robin to the 8 XCDs
// (each with its own L2); this gives every XCD one contiguous range of logical tile ids so
// neighbouring tiles (shared input halo, shared activation rows) meet in the same L2.
constexpr uint32_t xcd_remap(uint32_t bid, uint32_t nblocks) {
    const uint32_t per = nblocks >> 3, rem = nblocks & 7u;
    const uint32_t xcd = bid & 7u, idx = bid >> 3;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

// Tiles of workgroup b of a persistent grid of gx (a multiple of 8).  eighths: its XCD's contiguous eighth of the tiles, dealt to the
// XCD's workgroups in turn.  The kernels of a network that share this map (or xcd_remap's, which gives the same eighths) read most of
// what the kernel before them wrote from their own XCD's L2.  Measured by two plain kernels, a tensor written and read back with
// one map: 16 MB 6.6 us, 32 MB 9.7, 64 MB 21; every eighth read on another XCD than the one that wrote it: 13.9, 24.9, 31.  In the
// networks, whose kernels wait for other things as well, 1.4 to 1.8 % of ResNet50 at batch 256 (8-bit 1837 -> 1812 us, mixed 1816 -> 1783),
// nothing up to 192 (128 1035 and 1038, 192 1473 and 1475, 96 879 and 875; mixed at 96 and 128 and ResNet18 at 256 equal too).
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
// them and 1817 with a line of 65536; with a line of 38000, which takes in the 28 x 28 layers of batches up to 62, batch 52 603 and, here,
// 598, 56 620 and 615, 60 632 and 629; 104 to 240, in two parts, equal within 0.5 %).  One layer alone, above the line: the kernel
// with stages of a wave's own is 3 to 5 % faster in eighths, those with shared stages equal to 2 % slower.  conv1 + pool walks in
// eighths at every size (in turns the forward of batches 1 to 15 takes the same time, ResNet18 at 8 135.7 us, in eighths 135.1).
constexpr bool xcd_eighths(int64_t pixels) { return pixels >= 49152; }
// grid for it: at most `most` (a multiple of 8) workgroups, no more than the largest eighth needs
constexpr uint32_t xcd_walk_grid(int64_t n_tiles, uint32_t most) {
    const int64_t want = (n_tiles + 7) / 8 * 8;
    return want < most ? (uint32_t)want : most;
}

// The streaming 1x1 kernels' waves: n_ct channel tiles x `sequences` walks over the pixel groups, as many as fill the `slots` waves
// the chip holds at a time (rounded down: one workgroup past the last slot would be a round of its own).  even: a multiple of 8 of
// them, so that every XCD has whole sequences and as many as the others, where that gives up no more than a 33rd of them.
// Measured over 3400 shapes of 8192 to 200704 pixels, all sequences against a multiple of 8 (in turns below the line of the eighths,
// in eighths above it), operands in and out of the caches.  Kernel with stages of a wave's own, at most a 33rd given up: 1.4 % faster in
// turns, 3.1 in eighths (128 -> 192 at 94885 pixels 14.8 -> 12.7 us, 341 sequences and 336); more given up: 1.4 and 2.0 % slower (64 ->
// 832 + shortcut at 14884 11.7 us with 118, 14.0 with 112; 128 -> 416 + shortcut at 160152 54.1 with 157, 59.2 with 152).  Kernels with
// shared stages: nothing gained, and 3.3 and 6.1 % lost (256 -> 1408 + shortcut at 85227 69.7 with 46, 85 with 40).  They take all that
// fit (powers of two of channels make that an even number, which walks in eighths from the line on).
constexpr int32_t stream_sequences(int32_t slots, int32_t n_ct, int32_t n_groups, bool even) {
    const int32_t most = slots / n_ct, up = (n_groups + 7) / 8 * 8;
    if (most >= n_groups) return even && most >= up ? up : n_groups;      // (a group a wave; up: some have none)
    const int32_t n = most < 1 ? 1 : most, n8 = n / 8 * 8;
    return even && 33 * n8 >= 32 * n ? n8 : n;
}
// workgroups of four waves: an even launch's waves are counted within the XCD, the channel tiles of a sequence side by side
constexpr uint32_t stream_grid(int32_t n_ct, int32_t n_seq) {
    return n_seq % 8 == 0 ? ((uint32_t)(n_seq / 8) * n_ct + 3) / 4 * 8 : ((uint32_t)n_seq * n_ct + 3) / 4;
}
// spare: past the last sequence (of the XCD), nothing to do
struct StreamWave { int32_t ct; bool spare; TileWalk groups; };
constexpr StreamWave stream_wave(uint32_t b, uint32_t gx, int32_t wave, int32_t n_ct, int32_t n_seq, int32_t n_groups, bool eighths) {
    if ((n_seq & 7) == 0) {
        const int32_t g = (int32_t)(b >> 3) * 4 + wave, seq = g / n_ct;
        return {g - seq * n_ct, seq >= n_seq >> 3, xcd_walk((b & 7) | (uint32_t)seq << 3, (uint32_t)n_seq, n_groups, eighths)};
    }
    const int32_t g = (int32_t)xcd_remap(b, gx) * 4 + wave, seq = g / n_ct;
    return {g - seq * n_ct, seq >= n_seq, {seq, n_groups, n_seq}};
}

}  // namespace hawq
