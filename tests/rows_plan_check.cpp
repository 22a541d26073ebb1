// Walks the whole-row 3x3 kernel's plan over every output width on the host: the row division of every pixel a lane may ask
// for, and the LDS bytes that the pixel's window then reads; and the workgroups' tiles over every channel count: each tile
// exactly once, and evenly, in every grid.  Prints the first fault and returns 1, or the numbers of plans and grids taken.
#include <cstdio>
#include <vector>

#include "../paper_2011_10680_amd/csrc/conv3x3_rows_plan.h"

using namespace hawq;

int main() {
    const int heights[] = {1, 2, 3, 7, 16, 17, 56, 200};
    int taken = 0;
    for (int s2 = 0; s2 < 2; ++s2)
        for (int packed = 0; packed < 2; ++packed)
            for (int W = 1; W <= 2100; ++W)
                for (const int H : heights) {
                    const int P = s2 ? (H - 1) / 2 + 1 : H, Q = s2 ? (W - 1) / 2 + 1 : W;
                    RowsArgs g{};
                    if (!rows_plan(3, W, P, Q, s2, packed, g)) continue;
                    ++taken;
                    const int n_px = g.R * Q, pxb = packed ? 32 : 64;
                    const int rows = s2 ? 2 * g.R + 1 : g.R + 2;
                    bool ok = g.R >= 1 && g.R <= P && g.tpi * g.R >= P && (g.tpi - 1) * g.R < P && g.n_tiles == 3 * g.tpi && g.nt * 32 >= n_px &&
                              g.PW % (packed ? 32 : 16) == 0 && g.buf == rows * g.PW * pxb && 2 * g.buf <= 76 << 10;
                    for (int i = 0; ok && i < 32 * g.nt; ++i) {
                        const int ic = i < n_px ? i : n_px - 1, row = rows_row((uint32_t)ic, g.mq), q = ic - row * Q;
                        // stride 2: columns q and q + 1 of the even plane, q of the odd one; stride 1: columns q .. q + 2
                        const int last = s2 ? g.PWh + q : q + 2;
                        ok = row == ic / Q && q >= 0 && q < Q && last < g.PW && (!s2 || (q + 1 < g.PWh && g.PWh + q < 2 * g.PWh)) &&
                             ((s2 ? 2 * row : row) + 2) * g.PW + last < rows * g.PW;
                        if (!ok) std::printf("pixel %d (row %d, column %d): ", ic, row, q);
                    }
                    if (!ok) { std::printf("stride %d packed %d W %d H %d R %d\n", 1 + s2, packed, W, H, g.R); return 1; }
                }
    // every element offset below the marker 0x80000000, also those the kernel forms in 32 bits
    for (int64_t M = 1; M < ((int64_t)1 << 31); M = M * 3 / 2 + 1)
        for (int K = 64; K <= 65536; K *= 2)
            if (rows_offsets_fit(M, K) != ((uint64_t)M * (uint64_t)K - 1 < 0x7fffffffu)) { std::printf("M %lld K %d\n", (long long)M, K); return 1; }
    if (rows_offsets_fit((int64_t)1 << 25, 64) || !rows_offsets_fit(((int64_t)1 << 25) - 1, 64)) { std::printf("2^31 elements\n"); return 1; }
    int grids = 0;
    const int tile_counts[] = {1, 7, 8, 9, 20, 63, 126, 448, 896, 1793};
    for (int K = 64; K <= 70000; K += 64)
        for (const int n : tile_counts) {
            int32_t wc = 0, ncg = 0, gx = 0;
            if (!rows_grid(K, n, wc, ncg, gx)) continue;
            ++grids;
            std::vector<int> owners(n, 0);
            bool ok = gx > 0 && 32 * wc * ncg == K;
            // no workgroup has more tiles than an even division of an XCD's share gives its workgroups
            const int share = (n + 7) / 8, room = 512 / ncg / 8, per_xcd = room < 1 ? 1 : room < share ? room : share;
            const int most = (share + per_xcd - 1) / per_xcd;
            for (int b = 0; b < gx; ++b) {
                const RowsWalk w = rows_walk((uint32_t)b, (uint32_t)gx, n);
                ok = ok && w.step > 0 && w.first >= 0 && w.end <= n;
                int mine = 0;
                for (int t = w.first; ok && t < w.end; t += w.step, ++mine) ++owners[t];
                ok = ok && mine <= most;
            }
            for (int t = 0; t < n; ++t) ok = ok && owners[t] == 1;
            if (!ok) { std::printf("K %d: %d tiles on %d workgroups are not covered once each, or unevenly\n", K, n, gx); return 1; }
        }
    std::printf("%d plans %d grids\n", taken, grids);
    return 0;
}
