// Tiles of the whole-row 3x3 kernel (conv3x3_rows.hip): the arithmetic that its launcher and its device code share.  Plain C++
// (constexpr functions serve the host and the device), so that a program without a GPU can walk it over every size.
#pragma once
#include <stdint.h>

namespace hawq {

struct RowsArgs {
    int32_t R, tpi, n_tiles;      // output rows of a tile, tiles per image, tiles in all
    int32_t PW, PWh;              // pixels of an LDS row; stride 2: index of the first odd column in it
    int32_t nt;                   // MFMA column tiles (32 pixels) of a tile
    uint32_t mq;                  // i / Q for i < 32 nt: see rows_row
    int32_t buf;                  // bytes of one LDS buffer
};

// i / Q for an output pixel i of a tile, with mq = ceil(2^32 / Q).  Exact for Q >= 2 (i Q < 2^32); for Q = 1 the reciprocal
// does not fit 32 bits, rows_plan takes no such layer.
constexpr int rows_row(uint32_t i, uint32_t mq) { return (int)(((uint64_t)i * mq) >> 32); }

// Rows per tile and LDS layout for N images of W columns with P x Q outputs (s2: stride 2, else 1; packed: 4-bit operands);
// false: the kernel does not take the layer
constexpr bool rows_plan(int32_t N, int32_t W, int32_t P, int32_t Q, bool s2, bool packed, RowsArgs &g) {
    // a row of more than 1024 pixels fits no LDS buffer (and the byte counts below stay 32-bit)
    if (W > 1024 || Q < 2) return false;
    const int pxb = packed ? 32 : 64, al = packed ? 32 : 16;
    if (s2) {
        g.PWh = (Q + 1 + 15) / 16 * 16;                       // even columns -1, 1, ..., 2 Q - 1; as many odd ones, 0, 2, ...
        g.PW = (2 * g.PWh + al - 1) / al * al;
    } else {
        g.PWh = 0;
        g.PW = (W + 2 + al - 1) / al * al;
    }
    // the tile that wastes least: whole 32-pixel column tiles against R rows, rows against the image height
    double best = 0;
    g.R = 0;
    for (int R = 1; R <= 16 && R <= P; ++R) {
        const int rows = s2 ? 2 * R + 1 : R + 2;
        if (2 * rows * g.PW * pxb > (s2 ? 76 << 10 : 50 << 10)) break;
        const int tpi = (P + R - 1) / R, nt = (R * Q + 31) / 32;
        const double eff = (double)P * Q / ((double)tpi * nt * 32) * (nt >= 6 ? 1.0 : nt >= 4 ? 0.97 : 0.9);
        if (eff > best + 1e-9) { best = eff; g.R = R; g.tpi = tpi; g.nt = nt; g.buf = rows * g.PW * pxb; }
    }
    g.mq = (uint32_t)(((1ull << 32) + Q - 1) / Q);
    g.n_tiles = N * g.tpi;
    return g.R > 0;
}

// Element offsets of the output (and of the shortcut) stay below 2^31, the value that marks a pixel past the tile
constexpr bool rows_offsets_fit(int64_t M, int32_t K) { return M * K < ((int64_t)1 << 31); }

// Tiles of workgroup b of gx: first, first + step, ... below end.  Workgroup b runs on XCD b % 8, which owns a contiguous
// eighth of the tiles (rows shared by neighbours stay in its L2); its workgroups divide them.
struct RowsWalk { int32_t first, end, step; };
constexpr RowsWalk rows_walk(uint32_t b, uint32_t gx, int32_t n_tiles) {
    const uint32_t per = (uint32_t)(n_tiles + 7) / 8, xcd = b & 7;
    const uint32_t end = (xcd + 1) * per < (uint32_t)n_tiles ? (xcd + 1) * per : (uint32_t)n_tiles;
    return {(int32_t)(xcd * per + (b >> 3)), (int32_t)end, (int32_t)((gx + 7 - xcd) / 8)};
}

// Workgroups along the tiles (gx) for K output channels in groups of 32 wc: two workgroups per compute unit (registers), or
// one per tile.  A multiple of eight: every XCD then has as many workgroups as the others, and as its share has tiles (with one
// per tile and 238 tiles, two XCDs had 29 workgroups for 30 tiles: one tile's time more, 7.4 -> 10.0 us at 17 x 56 x 56).
// false: too many channel groups -- with fewer than eight workgroups an XCD's share has no owner.
constexpr bool rows_grid(int32_t K, int32_t n_tiles, int32_t &wc, int32_t &ncg, int32_t &gx) {
    wc = K % 128 == 0 ? 4 : 2;
    ncg = K / (32 * wc);
    gx = 512 / ncg / 8 * 8;
    if (gx > (n_tiles + 7) / 8 * 8) gx = (n_tiles + 7) / 8 * 8;
    return gx >= 8;
}

}  // namespace hawq
