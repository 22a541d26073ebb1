// Walks the input rows of every tile of the one-launch blocks over image sizes, batches and pixel sizes: a row's scalar offset lies
// inside the tensor, also for rows above and below the image, and is the row's own where the image has it.  Prints the first fault and
// returns 1, or the number of rows walked.
#include <cstdio>
#include <initializer_list>

#include "../paper_2011_10680_amd/csrc/conv_block_plan.h"

using namespace hawq;

int main() {
    long walked = 0;
    // (the last: an identity block's tensor just below 2^31 bytes)
    const int sizes[][3] = {{1, 1, 1}, {1, 3, 5}, {2, 7, 7}, {1, 8, 8}, {3, 9, 14}, {2, 16, 15}, {5, 25, 25}, {3, 33, 33}, {128, 56, 56}, {2, 57, 56}, {2674, 56, 56}};
    for (const auto &s : sizes)
        for (int bytes : {64, 128, 256}) {
            const int N = s[0], H = s[1], W = s[2];
            const long all = (long)N * H * W * bytes;
            for (int n = 0; n < N; ++n)
                for (int t = 0; t < (H + BLOCK_TH - 1) / BLOCK_TH; ++t)
                    for (int r = 0; r < BLOCK_HROWS; ++r, ++walked) {
                        const int y = t * BLOCK_TH - 1 + r;
                        const long at = block_input_row(n, y, H, W, bytes), own = ((long)n * H + y) * W * bytes;
                        const bool in = y >= 0 && y < H;
                        if (at < 0 || at + (long)W * bytes > all || (in && at != own)) {
                            std::printf("row %d of image %d of %d x %d x %d: offset %ld of %ld\n", y, n, N, H, W, at, all);
                            return 1;
                        }
                    }
        }
    std::printf("%ld\n", walked);
    return 0;
}
