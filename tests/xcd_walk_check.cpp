// Walks every workgroup's tiles over many tile counts and grids: each tile exactly once, eighths in order, no workgroup more than
// one round ahead of its XCD's others.  Prints the first fault and returns 1, or the number of grids walked.
#include <cstdio>
#include <vector>

#include "../paper_2011_10680_amd/csrc/xcd_walk.h"

using namespace hawq;

int main() {
    int walked = 0;
    for (int n = 1; n < 6000; n += n < 600 ? 1 : 37)
        for (uint32_t most : {8u, 64u, 336u, 512u, 768u, 2048u}) {
            const uint32_t gx = xcd_walk_grid(n, most);
            if (gx < 8 || gx % 8 != 0 || gx > most) { std::printf("grid %u of at most %u for %d tiles\n", gx, most, n); return 1; }
            std::vector<int> owner(n, -1);
            for (uint32_t b = 0; b < gx; ++b) {
                const TileWalk w = xcd_walk(b, gx, n);
                int rounds = 0;
                for (int t = w.first; t < w.end; t += w.step, ++rounds) {
                    if (t < 0 || t >= n || owner[t] != -1) { std::printf("tile %d of %d, workgroup %u of %u\n", t, n, b, gx); return 1; }
                    owner[t] = (int)(b & 7);
                }
                if (rounds > (n / 8 + 1 + (int)gx / 8 - 1) / ((int)gx / 8)) { std::printf("%d rounds: %d tiles, workgroup %u of %u\n", rounds, n, b, gx); return 1; }
            }
            for (int t = 0; t < n; ++t)
                if (owner[t] < 0 || (t > 0 && owner[t] < owner[t - 1])) { std::printf("tile %d of %d, grid %u\n", t, n, gx); return 1; }
            std::vector<int> turns(n, 0);   // the other map: each tile once, in as many rounds
            for (uint32_t b = 0; b < gx; ++b) {
                const TileWalk w = xcd_walk(b, gx, n, false);
                for (int t = w.first; t < w.end; t += w.step)
                    if (t < 0 || t >= n || turns[t]++ != 0) { std::printf("turns: tile %d of %d, workgroup %u of %u\n", t, n, b, gx); return 1; }
            }
            for (int t = 0; t < n; ++t)
                if (turns[t] != 1) { std::printf("turns: tile %d of %d, grid %u\n", t, n, gx); return 1; }
            ++walked;
        }
    std::printf("%d\n", walked);
    return 0;
}
