// The shortcut of a byte in floating point as the one-launch blocks compute it, against the shifted sum: every byte, every shift that a
// network admits there, multipliers at random, at the ends of their range and where the products meet a half.  Prints the first fault
// and returns 1, or the number of terms compared.
#include <cstdio>
#include <random>
#include <vector>

#include "../paper_2011_10680_amd/csrc/conv_block_plan.h"

using namespace hawq;

int main() {
    if (res_float_ok(65536, 8) || res_float_ok(8, 1) || !res_float_ok(65535, 2) || !res_float_ok(0, 62)) { std::printf("range\n"); return 1; }
    std::mt19937 g(5);
    long compared = 0;
    for (int rc = 2; rc <= 30; ++rc) {
        std::vector<int32_t> rbs = {0, 1, 2, 3, 16384, 32767, 32768, 32769, 65534, 65535};
        for (int k = 0; k < 16; ++k) for (int d = -1; d <= 1; ++d) rbs.push_back(((1 << k) + d) & 65535);
        for (int k = 0; k < 3000; ++k) rbs.push_back((int32_t)(g() & 65535));
        for (const int32_t rb : rbs) {
            const int32_t rf = res_float(rb, rc);
            for (int r = 0; r < 256; ++r, ++compared) {
                const int32_t want = (int32_t)(((int64_t)r * rb + (1ll << (rc - 1))) >> rc), got = res_scaled((float)r, rf) - kResMagic;
                if (got != want) { std::printf("%d * %d >> %d: %d, not %d\n", r, rb, rc, got, want); return 1; }
            }
        }
    }
    std::printf("%ld\n", compared);
    return 0;
}
