// First layer of the networks: 7x7 stride-2 pad-3 convolution of a 3-channel uint8 image to 64
// channels (Appendix H keeps this layer at 8 bits), on the INT8 matrix cores.
//
// The image holds 0..255, which does not fit the signed INT8 operand.  The kernel feeds x - 128
// (x XOR 0x80) and the host adds 128 * sum(w[k]) to the bias; out-of-image taps are filled with
// raw 0, i.e. -128 after the offset, so the correction is the same at every pixel.  Exact.
//
// K layout: pixels are widened to 4 bytes (RGB0) while staging, a filter row becomes 8 pixels x
// 4 bytes = 32 bytes = one 32x32x32 MFMA K-step, and the 7 rows plus one zero row give K = 256.
// Weights arrive re-tiled by the host as [64][8][8][4] with zeros in the padding positions.
// A workgroup computes a 16x16 tile of output pixels for all 64 channels from a 37x40-pixel
// input patch staged once in LDS; each input byte is read from HBM once per workgroup.
#include "common.h"
#include "epilogue.h"

namespace hawq {

constexpr int STEM_TILE = 16;                    // output tile edge
constexpr int STEM_ROWS = 2 * STEM_TILE + 5;     // 37 input rows
constexpr int STEM_COLS = 40;                    // patch width in pixels (38 used), origin = 2*q0 - 3
constexpr int STEM_W_BYTES = 64 * 256;

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) conv_stem_kernel(const ConvArgs a, const int tiles_q, const int tiles_p) {
    __shared__ __attribute__((aligned(16))) uint8_t lw[STEM_W_BYTES];
    __shared__ __attribute__((aligned(16))) uint32_t lx[STEM_ROWS * STEM_COLS];
    __shared__ ChanMain par_m[64];
    __shared__ ChanRes par_r[64];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int bid = blockIdx.x;
    const int tq = bid % tiles_q; bid /= tiles_q;
    const int tp_ = bid % tiles_p;
    const int n = bid / tiles_p;
    const int p0 = tp_ * STEM_TILE, q0 = tq * STEM_TILE;

    // ---- stage weights: 1024 16-byte chunks, swizzled by channel ----
    for (int i = tid; i < STEM_W_BYTES / 16; i += 256) {
        const int row = i >> 4, ch = i & 15;
        *(v4i *)(lw + row * 256 + ((ch ^ (row & 15)) << 4)) = *(const v4i *)(a.w + i * 16);
    }
    // ---- stage the input patch: groups of 4 pixels (12 bytes, dword aligned) -> 4 RGB0 dwords ----
    const uint8_t *img = a.x + (int64_t)n * a.H * a.W * 3;
    for (int i = tid; i < STEM_ROWS * 10; i += 256) {
        const int rl = i / 10, g = i - rl * 10;
        const int ih = 2 * p0 - 3 + rl;
        const int iw = 2 * q0 - 4 + 4 * g;       // first pixel of the group; patch column = 4g - 1
        uint32_t px[4] = {0, 0, 0, 0};
        if ((unsigned)ih < (unsigned)a.H && iw >= 0 && iw + 3 < a.W) {
            const uint32_t *src = (const uint32_t *)(img + ((int64_t)ih * a.W + iw) * 3);
            const uint32_t d0 = src[0], d1 = src[1], d2 = src[2];
            px[0] = d0 & 0x00ffffffu;
            px[1] = ((d0 >> 24) | (d1 << 8)) & 0x00ffffffu;
            px[2] = ((d1 >> 16) | (d2 << 16)) & 0x00ffffffu;
            px[3] = d2 >> 8;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int col = 4 * g - 1 + k;
            if (col >= 0 && col < STEM_COLS) lx[rl * STEM_COLS + col] = px[k] ^ 0x00808080u;
        }
    }
    const bool tile_epi = a.y_dt != HAWQ_S32;
    int wide = 0;
    if (tile_epi) wide = stage_params(a, 0, 64, par_m, par_r);
    wide = __syncthreads_or(wide);

    // ---- MFMA: wave w owns output rows 4w..4w+3 of the tile (2 pixel tiles of 2 rows x 16 cols) ----
    const int rho = lane & 31, khalf = lane >> 5;
    const int hsel = (rho >> 2) & 1, isel = (rho >> 3) * 4 + (rho & 3);
    int a_row[2];
#pragma unroll
    for (int tc = 0; tc < 2; ++tc) a_row[tc] = hsel * 32 + tc * 16 + isel;
    int b_base[2];
#pragma unroll
    for (int tp = 0; tp < 2; ++tp) {
        const int pr = wave * 4 + tp * 2 + (rho >> 4), pc = rho & 15;
        b_base[tp] = (2 * pr) * STEM_COLS + 2 * pc + 4 * khalf;   // dword index; K-step r adds r*STEM_COLS
    }
    v16i acc[2][2];
#pragma unroll
    for (int tp = 0; tp < 2; ++tp)
#pragma unroll
        for (int tc = 0; tc < 2; ++tc)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tp][tc][i] = 0;

#pragma unroll
    for (int r = 0; r < 7; ++r) {   // the 8th K-step multiplies zero weights: skipped
        v4i af[2], bf[2];
#pragma unroll
        for (int tc = 0; tc < 2; ++tc) {
            const int row = a_row[tc];
            af[tc] = *(const v4i *)(lw + row * 256 + (((2 * r + khalf) ^ (row & 15)) << 4));
        }
#pragma unroll
        for (int tp = 0; tp < 2; ++tp) {
            const uint2 lo = *(const uint2 *)(lx + b_base[tp] + r * STEM_COLS);
            const uint2 hi = *(const uint2 *)(lx + b_base[tp] + r * STEM_COLS + 2);
            bf[tp] = (v4i){(int)lo.x, (int)lo.y, (int)hi.x, (int)hi.y};
        }
#pragma unroll
        for (int tp = 0; tp < 2; ++tp)
#pragma unroll
            for (int tc = 0; tc < 2; ++tc)
                acc[tp][tc] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[tc], bf[tp], acc[tp][tc], 0, 0, 0);
    }

    const int ch0 = khalf * 32;
    if (tile_epi) {
        int64_t mm[2];
        bool valid[2];
#pragma unroll
        for (int tp = 0; tp < 2; ++tp) {
            const int p = p0 + wave * 4 + tp * 2 + (rho >> 4), q = q0 + (rho & 15);
            valid[tp] = p < a.P && q < a.Q;
            mm[tp] = ((int64_t)n * a.P + p) * a.Q + q;
        }
        const uint32_t none[2][2][4] = {};
        epilogue_tile<2, 2, false>(a, par_m, par_r, mm, valid, 0, ch0, acc, wide, none);
        return;
    }
    static_for<0, 2>([&](auto tpc) {
        constexpr int tp = decltype(tpc)::value;
        const int p = p0 + wave * 4 + tp * 2 + (rho >> 4), q = q0 + (rho & 15);
        if (p >= a.P || q >= a.Q) return;
        const int64_t m = ((int64_t)n * a.P + p) * a.Q + q;
        epilogue_pixel<2, true>(a, m, ch0, acc[tp]);
    });
}

// ---------------------------------------------------------------------------------------------------
// conv1 fused with the 3x3/2 max pool that follows it in every ResNet: the conv1 tensor (the largest of the network) is
// never written to or read from HBM -- and never requantised either.  Requantisation (Section 3.1) and the clamps are
// non-decreasing in the accumulator for every multiplier the interface admits (b >= 0), so the maximum commutes with
// them exactly: the kernel takes the maximum over a window's INT32 accumulators (+ the channel's bias, the same for every
// pixel) and requantises once per *pooled* output, 4.5 times fewer 64-bit multiplies than conv1 has outputs.
//
// For that a pooling window's nine accumulators must meet in one lane.  The MFMA leaves a lane with one column and
// sixteen rows of the 32x32 result, so here the *pixels* are the row operand and the channels the column operand (the
// other way round from every other kernel of the library): lane (n, h) ends up with channel n and the sixteen pixels in
// rows {8j + 4h + q}.  Which conv1 pixel feeds which row is the kernel's choice: the 48 rows that a lane half has in three
// MFMA tiles hold a block of 5 x 9 conv1 outputs (three slots spare) -- the windows of 2 x 4 pooled pixels.  6 slots a
// pooled pixel, where 9 conv1 outputs without sharing and 4 at best would be needed, and one MFMA tile alone, 3 x 5 outputs
// for two pooled pixels, took 8.
//
// What bounds it: the matrix pipes have 42 instructions for 16 pooled pixels of 64 channels, 14 us at batch 128 (224 x 224); the
// image and the pooled tensor are 45 MB, 9 us.  56 -> 41 us at batch 128, 102 -> 70 at 256, 30 -> 24 at 64, 7.9 and 8.0 at
// batch 1 against a tile of 3 x 5 conv1 outputs at a time (14 instructions for four pooled pixels; three waves on a SIMD where
// this has two).  Of that 45 us came with the larger block, 3 with fragment reads free of bank conflicts, branch-free loads and
// places in the image that are stepped and not divided.  Matrix pipes 40 %, vector ALU 30 %, LDS half of the cycles (a quarter
// of the LDS's are still conflicts, of the staging's and the results' writes): what is left is each wave's own chain of multiplying,
// taking maxima and staging, with two of them on a SIMD to overlap.
//
// A workgroup (four waves) makes 8 x 8 tiles of pooled pixels from a 39 x 41 input patch staged in LDS (pixels widened to
// RGB0 dwords; a filter row = 8 pixels x 4 B = one K = 32 MFMA step), two pooled rows to a wave: the addresses of a lane's
// row operands are the same for every tile.  The 64 x 7 x 32 weight bytes a lane needs as column operand (two channels)
// stay in registers for the life of the (persistent) workgroup.  Results go through an LDS tile to become 16-byte NHWC
// stores.  Patch and result tile have two places each: one barrier a tile, behind which a wave stores its share of this
// tile and goes on to the next.
constexpr int FUSE_PT = 8;                         // pooled tile edge
constexpr int FUSE_CT = 2 * FUSE_PT + 1;           // 17 conv rows / columns under it
constexpr int FUSE_ROWS = 2 * FUSE_CT + 5;         // 39 input rows
// The patch is 41 pixels wide (origin = image column 4*pq0 - 5), its rows in pairs of 98 dwords, the second of a pair 48 behind the
// first: the 32 lanes of one pass of a fragment read touch parts of up to three conv1 rows (a pair each), 34 consecutive dwords a
// whole row, and 98 = 34 (mod 64 banks) lays them side by side without an overlap in all three tiles (rows of 48: an overlap of
// two dwords in each pass, every one two cycles)
constexpr int FUSE_PAIR = 98, FUSE_ODD = 48;
constexpr int FUSE_PATCH = (FUSE_ROWS + 1) / 2 * FUSE_PAIR + 4;   // (four dwords before the first row, which staging may write)
constexpr int FUSE_PITCH = 80;                     // bytes of a pooled pixel in LDS (64: both lane halves in the same banks)
constexpr int FUSE_GROUPS = 11;                    // 4-pixel groups fetched per patch row (patch columns -3 .. 40)

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
conv_stem_pool_kernel(const ConvArgs a, const int pool_P, const int pool_Q, const int pool_y_dt, const int pool_lo,
                      const int pool_hi, uint8_t *__restrict__ pool_y, const int tiles_q, const int tiles_p, const int n_tiles) {
    __shared__ __attribute__((aligned(16))) uint32_t lx[2][FUSE_PATCH];
    __shared__ __attribute__((aligned(16))) uint8_t lp[2][FUSE_PT * FUSE_PT * FUSE_PITCH];   // pooled tile [row][column][channel]
    __shared__ ChanMain par_m[64];
    __shared__ ChanRes par_r[64];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    // input patch of a tile: row rl <-> image row 4*pp0 - 5 + rl, column c <-> image column 4*pq0 - 5 + c; groups of 4
    // pixels (12 bytes) start at image column 4*pq0 - 8 + 4g, i.e. patch column 4g - 3.  A thread owns work items tid
    // and tid + 256 of the FUSE_ROWS * FUSE_GROUPS groups.
    constexpr int NITEM = (FUSE_ROWS * FUSE_GROUPS + 255) / 256;
    // (items beyond the last and the first three columns of a row's first group go to places that nobody reads)
    const int row_bytes = a.W * 3;
    int it_row[NITEM], it_col[NITEM], it_off[NITEM];
    uint32_t *it_dst[NITEM];
#pragma unroll
    for (int it = 0; it < NITEM; ++it) {
        const int i = tid + it * 256, rl = i / FUSE_GROUPS, g = i - rl * FUSE_GROUPS;
        it_row[it] = rl < FUSE_ROWS ? rl - 5 : -(1 << 30);        // (a row that no image has)
        it_col[it] = 4 * g - 8;
        it_off[it] = rl * row_bytes + 12 * g;
        const int to = min(rl, FUSE_ROWS);
        it_dst[it] = &lx[0][4] + (to >> 1) * FUSE_PAIR + (to & 1) * FUSE_ODD + 4 * g - 3;
    }
    typedef uint32_t v3u __attribute__((ext_vector_type(3)));
    v3u raw[NITEM];
    const TileWalk walk = xcd_walk(blockIdx.x, gridDim.x, n_tiles);
    // a tile's place: column, row of its image, image; and what a step of the walk adds
    struct Place { int q, p, n; };
    auto place = [&](int tile) { Place c; c.q = tile % tiles_q; tile /= tiles_q; c.p = tile % tiles_p; c.n = tile / tiles_p; return c; };
    const Place step = place(walk.step);
    auto advance = [&](Place c) {
        c.q += step.q; c.p += step.p; c.n += step.n;
        if (c.q >= tiles_q) { c.q -= tiles_q; ++c.p; }
        if (c.p >= tiles_p) { c.p -= tiles_p; ++c.n; }
        return c;
    };
    auto fetch = [&](const Place &c) {
        // (offsets from the patch's first group, which may lie outside the image: every lane that does reads zeros)
        const int y0 = 4 * c.p * FUSE_PT, x0 = 4 * c.q * FUSE_PT;
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)(a.x + (((int64_t)c.n * a.H + y0 - 5) * a.W + x0 - 8) * 3), 0, 0x7fffffff, 0x00020000);
#pragma unroll
        for (int it = 0; it < NITEM; ++it) {
            const bool in = ((unsigned)(y0 + it_row[it]) < (unsigned)a.H) & ((unsigned)(x0 + it_col[it]) < (unsigned)a.W);   // (a.W is a multiple of 4, so is a group's column)
            raw[it] = __builtin_amdgcn_raw_buffer_load_b96(rx, in ? it_off[it] : (int)0x80000000u, 0, 0);
        }
    };
    // widen the fetched RGB triples to RGB0 dwords, offset by -128 (XOR 0x80 per byte), into the LDS patch;
    // out-of-image positions are raw zeros and get the same offset (the bias correction assumes it everywhere)
    auto stage = [&](int to) {
#pragma unroll
        for (int it = 0; it < NITEM; ++it) {
            const uint32_t d0 = raw[it][0], d1 = raw[it][1], d2 = raw[it][2];
            uint32_t *dst = it_dst[it] + to * FUSE_PATCH;
            dst[0] = (d0 & 0x00ffffffu) ^ 0x00808080u;
            dst[1] = (__builtin_amdgcn_alignbyte(d1, d0, 3) & 0x00ffffffu) ^ 0x00808080u;
            dst[2] = (__builtin_amdgcn_alignbyte(d2, d1, 2) & 0x00ffffffu) ^ 0x00808080u;
            dst[3] = (d2 >> 8) ^ 0x00808080u;
        }
    };
    // (the first tile's bytes are under way while the parameters come)
    if (walk.first >= walk.end) return;    // (the whole workgroup)
    int tile = walk.first;
    Place cur = place(tile), nxt = advance(cur);
    fetch(cur);
    int wide = stage_params(a, 0, 64, par_m, par_r);
    wide = __syncthreads_or(wide);
    // column operand: channel col + 32 tc, K-step r (filter row), this lane half's 16 bytes (filter columns 4 half .. + 3)
    v4i wf[7][2];
#pragma unroll
    for (int r = 0; r < 7; ++r)
#pragma unroll
        for (int tc = 0; tc < 2; ++tc) wf[r][tc] = *(const v4i *)(a.w + (((col + 32 * tc) * 8 + r) * 8 + 4 * half) * 4);
    // row operand: MFMA row rho of tile mt is slot 16 mt + 4 (rho >> 3) + (rho & 3) of the block of lane half (rho >> 2) & 1;
    // slot s < 45 is conv1 pixel (s / 9, s % 9) of the 5 x 9 block (the rest repeat slot 44 and are never looked at)
    int bb[3];
#pragma unroll
    for (int mt = 0; mt < 3; ++mt) {
        const int s = min(16 * mt + 4 * (col >> 3) + (col & 3), 44), br = s / 9, bc = s - 9 * br;
        bb[mt] = 4 + (4 * wave + br) * FUSE_PAIR + 2 * (8 * ((col >> 2) & 1) + bc) + 4 * half;
    }
    // the convolution's clamp and the pool's as one
    int32_t lo_c = min(max(a.lo, pool_lo), pool_hi), hi_c = min(max(a.hi, pool_lo), pool_hi);
    asm volatile("" : "+v"(lo_c), "+v"(hi_c));

    const uint32_t st_off = (uint32_t)(((tid >> 5) * pool_Q + (tid >> 2 & 7)) * 64 + (tid & 3) * 16);   // a thread's pixel and channels in the pooled tensor

    auto run = [&](auto wide_c) {
        int buf = 0;
        stage(0);
        if (tile + walk.step < walk.end) fetch(nxt);
        __syncthreads();
        for (;;) {
            const int pp0 = cur.p * FUSE_PT, pq0 = cur.q * FUSE_PT;       // pooled tile origin
            v16i acc[3][2];
            {
                const uint32_t *patch = lx[buf];
                auto frag = [&](int r, int mt) {
                    const uint32_t *p = patch + bb[mt] + (r >> 1) * FUSE_PAIR + (r & 1) * FUSE_ODD;
                    const uint2 l0 = *(const uint2 *)p;
                    const uint2 h0 = *(const uint2 *)(p + 2);
                    return (v4i){(int)l0.x, (int)l0.y, (int)h0.x, (int)h0.y};
                };
                v4i pf[2][3];
#pragma unroll
                for (int mt = 0; mt < 3; ++mt) pf[0][mt] = frag(0, mt);
#pragma unroll
                for (int r = 0; r < 7; ++r) {   // the 8th K-step multiplies zero weights: skipped
                    if (r < 6)
#pragma unroll
                        for (int mt = 0; mt < 3; ++mt) pf[(r + 1) & 1][mt] = frag(r + 1, mt);
#pragma unroll
                    for (int mt = 0; mt < 3; ++mt)
#pragma unroll
                        for (int tc = 0; tc < 2; ++tc)
                            acc[mt][tc] = __builtin_amdgcn_mfma_i32_32x32x32_i8(pf[r & 1][mt], wf[r][tc], r == 0 ? (v16i){} : acc[mt][tc], 0, 0, 0);
                }
            }
            const int next = tile + walk.step;
            const bool more = next < walk.end;
            const Place after = advance(nxt);
            if (more) {
                stage(buf ^ 1);
                if (next + walk.step < walk.end) fetch(after);
            }
            // ---- this lane: channels col, col + 32; pooled pixels (2 wave + 0..1, 4 half + 0..3) of the tile ----
            auto at = [&](int tc, int r, int c) -> int32_t { return acc[(9 * r + c) / 16][tc][(9 * r + c) % 16]; };
            // taps outside the image do not take part: rows are the same for the wave, columns for a lane half
            const int cr0 = 2 * (pp0 + 2 * wave) - 1;                // conv1 row of the block's first
            if (cr0 < 0 || cr0 + 4 >= a.P)
#pragma unroll
            for (int r = 0; r < 5; ++r)
                if ((unsigned)(cr0 + r) >= (unsigned)a.P)
#pragma unroll
                    for (int s = 9 * r; s < 9 * r + 9; ++s) acc[s / 16][0][s % 16] = acc[s / 16][1][s % 16] = INT32_MIN;
            if (cur.q == 0 || 2 * (pq0 + FUSE_PT) > a.Q) {
                const int cq0 = 2 * (pq0 + 4 * half) - 1;
#pragma unroll
                for (int c = 0; c < 9; ++c) {
                    const bool in = (unsigned)(cq0 + c) < (unsigned)a.Q;
#pragma unroll
                    for (int s = c; s < 45; s += 9)
#pragma unroll
                        for (int tc = 0; tc < 2; ++tc) acc[s / 16][tc][s % 16] = in ? acc[s / 16][tc][s % 16] : INT32_MIN;
                }
            }
            uint8_t *out = lp[buf] + (2 * wave * FUSE_PT + 4 * half) * FUSE_PITCH + col;
#pragma unroll
            for (int tc = 0; tc < 2; ++tc) {
                // the channel's requantisation: narrow form  high word of t * bs + Rs  (bias inside Rs), else the exact 64-bit form
                const ChanMain &q = par_m[col + 32 * tc];
                int32_t m[5][4];           // maxima over a row's three columns
#pragma unroll
                for (int r = 0; r < 5; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) m[r][c] = max(max(at(tc, r, 2 * c), at(tc, r, 2 * c + 1)), at(tc, r, 2 * c + 2));
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const int32_t mm = max(max(m[2 * r][c], m[2 * r + 1][c]), m[2 * r + 2][c]);
                        int32_t y;
                        // (wrapping sum: a pooled pixel outside the tensor carries INT32_MIN and is never stored)
                        if (decltype(wide_c)::value) y = clamp64(rq64((int32_t)((uint32_t)mm + (uint32_t)q.bias), q.b, q.c), lo_c, hi_c);
                        else {
                            const int32_t v = (int32_t)(((int64_t)mm * (int64_t)q.bs + q.Rs) >> 32);
                            asm("v_med3_i32 %0, %1, %2, %3" : "=v"(y) : "v"(v), "v"(lo_c), "v"(hi_c));
                        }
                        out[(r * FUSE_PT + c) * FUSE_PITCH + 32 * tc] = (uint8_t)y;
                    }
            }
            __syncthreads();              // pooled tile and the next patch complete

            // ---- 16 channels of one pooled pixel per thread: 16-byte NHWC stores ----
            if (pp0 + (tid >> 5) < pool_P && pq0 + (tid >> 2 & 7) < pool_Q) {
                const uint4 v = *(const uint4 *)(lp[buf] + (tid >> 2) * FUSE_PITCH + (tid & 3) * 16);
                const int64_t oe = (((int64_t)cur.n * pool_P + pp0) * pool_Q + pq0) * 64;
                if (is4(pool_y_dt)) {
                    // low nibbles of the four bytes of a dword -> 16 bits (values <= 15 by the clamp)
                    auto nib = [](uint32_t d) { return (d & 0xfu) | ((d >> 4) & 0xf0u) | ((d >> 8) & 0xf00u) | ((d >> 12) & 0xf000u); };
                    *(uint2 *)(pool_y + (oe >> 1) + (st_off >> 1)) = make_uint2(nib(v.x) | (nib(v.y) << 16), nib(v.z) | (nib(v.w) << 16));
                } else {
                    *(uint4 *)(pool_y + oe + st_off) = v;
                }
            }
            if (!more) break;
            tile = next;
            cur = nxt; nxt = after;
            buf ^= 1;
        }
    };
    if (wide) run(std::true_type{});
    else run(std::false_type{});
}

hawq_status launch_conv_stem_pool(const ConvArgs &a, int pool_y_dt, int pool_lo, int pool_hi, void *pool_y, hipStream_t s) {
    if (a.M == 0) return HAWQ_OK;
    const int pool_P = (a.P - 1) / 2 + 1, pool_Q = (a.Q - 1) / 2 + 1;
    const int tiles_p = (pool_P + FUSE_PT - 1) / FUSE_PT, tiles_q = (pool_Q + FUSE_PT - 1) / FUSE_PT;
    const int64_t n_tiles = (int64_t)a.N * tiles_p * tiles_q;
    if (n_tiles > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
    const uint32_t grid = xcd_walk_grid(n_tiles, 2 * 256);         // persistent: two workgroups per CU
    // the pooled bytes are unsigned: bounds outside 0..255 never bind
    pool_lo = pool_lo < 0 ? 0 : pool_lo;
    pool_hi = pool_hi > 255 ? 255 : pool_hi;
    conv_stem_pool_kernel<<<grid, 256, 0, s>>>(a, pool_P, pool_Q, pool_y_dt, pool_lo, pool_hi, (uint8_t *)pool_y,
                                                          tiles_q, tiles_p, (int)n_tiles);
    return check_launch();
}

// Re-tile [64][7][7][3] int8 weights to [64][8][8][4] (zeros in the padding) -- host helper.
void stem_pack_weights(const int8_t *w, int8_t *out) {
    for (int k = 0; k < 64; ++k)
        for (int r = 0; r < 8; ++r)
            for (int s = 0; s < 8; ++s)
                for (int c = 0; c < 4; ++c)
                    out[((k * 8 + r) * 8 + s) * 4 + c] = (r < 7 && s < 7 && c < 3) ? w[((k * 7 + r) * 7 + s) * 3 + c] : 0;
}

bool conv_stem_eligible(const ConvArgs &a) {
    return a.C == 3 && a.K == 64 && a.R == 7 && a.S == 7 && a.stride_h == 2 && a.stride_w == 2 && a.pad_h == 3 &&
           a.pad_w == 3 && a.x_dt == HAWQ_U8 && a.w_dt == HAWQ_S8 && a.W % 4 == 0 && a.res == nullptr && a.b != nullptr &&
           (((uintptr_t)a.x | (uintptr_t)a.w | (uintptr_t)a.y | (uintptr_t)a.bias | (uintptr_t)a.b) & 15) == 0 &&
           ((uintptr_t)a.c & 3) == 0;
}

hawq_status launch_conv_stem(const ConvArgs &a, hipStream_t s) {
    if (a.M == 0) return HAWQ_OK;
    const int tiles_p = (a.P + STEM_TILE - 1) / STEM_TILE, tiles_q = (a.Q + STEM_TILE - 1) / STEM_TILE;
    const int64_t blocks = (int64_t)a.N * tiles_p * tiles_q;
    if (blocks > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
    conv_stem_kernel<<<(uint32_t)blocks, 256, 0, s>>>(a, tiles_q, tiles_p);
    return check_launch();
}

}  // namespace hawq
