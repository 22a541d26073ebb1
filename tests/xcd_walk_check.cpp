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
    // the streaming kernels' waves: every group of every channel tile once, with all the sequences the slots hold or, even,
    // a 33rd fewer, and no more waves than there are slots
    for (int n = 100; n < 7000; n += n < 700 ? 21 : 701)
        for (int n_ct = 1; n_ct < 300; n_ct += n_ct < 70 ? 1 : 23)
            for (int slots : {2048, 3072, 4096})
                for (int form = 0; form < 4; ++form) {
                    const bool even = form & 1, eighths = form & 2;
                    const int n_seq = stream_sequences(slots, n_ct, n, even);
                    const uint32_t gx = stream_grid(n_ct, n_seq);
                    const int most = slots / n_ct < n ? slots / n_ct : n;
                    int turns = 0, spares = 0;
                    std::vector<int> done((size_t)n * n_ct, 0);
                    for (uint32_t b = 0; b < gx; ++b)
                        for (int wave = 0; wave < 4; ++wave) {
                            const StreamWave w = stream_wave(b, gx, wave, n_ct, n_seq, n, eighths);
                            int t = 0;
                            if (w.spare) { ++spares; continue; }
                            for (int g = w.groups.first; g < w.groups.end; g += w.groups.step, ++t)
                                if (w.ct < 0 || w.ct >= n_ct || g < 0 || g >= n || done[(size_t)g * n_ct + w.ct]++ != 0) {
                                    std::printf("group %d of %d, channel tile %d of %d, %d sequences\n", g, n, w.ct, n_ct, n_seq);
                                    return 1;
                                }
                            turns = t > turns ? t : turns;
                        }
                    for (int d : done)
                        if (d != 1) { std::printf("%d groups, %d channel tiles, %d sequences: one is missing\n", n, n_ct, n_seq); return 1; }
                    const int fewest = even && most < n ? (32 * most + 32) / 33 : most;
                    if (n_seq < fewest || (even && fewest % 8 == 0 && n_seq % 8 != 0) || turns > (n + fewest - 1) / fewest + (even ? 1 : 0) || (n_ct % 4 == 0 && spares != 0) || n_seq * n_ct > slots) {
                        std::printf("%d groups, %d channel tiles, %d sequences: %d turns, %d spare waves\n", n, n_ct, n_seq, turns, spares);
                        return 1;
                    }
                    // a workgroup's waves share their walk where the channel tiles come in fours: its barriers meet
                    if (n_ct % 4 == 0)
                        for (uint32_t b = 0; b < gx; ++b)
                            for (int wave = 1; wave < 4; ++wave) {
                                const StreamWave v = stream_wave(b, gx, 0, n_ct, n_seq, n, eighths), w = stream_wave(b, gx, wave, n_ct, n_seq, n, eighths);
                                if (v.groups.first != w.groups.first || v.groups.end != w.groups.end) { std::printf("workgroup %u: two walks\n", b); return 1; }
                            }
                    ++walked;
                }
    std::printf("%d\n", walked);
    return 0;
}
