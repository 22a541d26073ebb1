// 3x3 convolution with 64 input channels, stride 1 or 2, on whole output rows: weights resident in registers, pixels in LDS
// with their zero padding written out.
//
// The 64-channel 3x3 layers (stage 1 of the networks, the first down-sampling layer) have the lowest arithmetic intensity
// of all, so everything around the MFMAs shows.  What conv3x3_c64.hip spends beside them: its weight fragments come from LDS
// for every tile (36 of 54 fragment reads), and a tile of consecutive pixels makes every lane find out, per tile and per
// tap, whether its pixel's tap lies inside the image.  Here:
//   * a wave keeps the 18 weight fragments of its 32 output channels in registers for its whole life (72 VGPRs) and walks
//     tiles; only pixel fragments are read from LDS, one per MFMA;
//   * a tile is R whole output rows of one image, and LDS holds the input rows under them with a column of zeros on each
//     side (and rows of zeros above and below the image): no tap is ever outside, a lane's addresses depend on its position
//     in the tile only, and output pixels of a tile are consecutive in memory.  The LDS-DMA that fetches the rows writes the
//     zeros by itself (out-of-range offsets);
//   * an LDS row is PW pixels long, a multiple of 16, so that a row step leaves the chunk permutation alone (pixel p keeps
//     chunk c at c ^ (p >> 2): sixteen consecutive pixels of one LDS row lie in sixteen different banks; a column tile that
//     crosses a row end continues PW - Q pixels further, 8 of 16 for 56 columns, and collides: 0.20 to 0.33 of the LDS-active
//     cycles are conflicts there).  Stride 2 keeps the even columns of a row before the odd ones, so that a tap's pixels are
//     consecutive again.
// Two buffers of rows: the next tile's are fetched while this one is multiplied, one barrier per tile.
// PK: packed 4-bit operands; pixels stay packed in LDS (32 bytes), a lane takes its half's nibbles on the way into the MFMA.
#include "conv3x3_rows_plan.h"
#include "rp.h"

namespace hawq {

// WC: channel groups of 32 (waves along channels), 4 / WC waves along pixels.
template <int WC, bool S2, bool PK, bool RES>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) conv3x3_rows_kernel(const ConvArgs a, const RowsArgs g) {
    constexpr int WP = 4 / WC, KG = 32 * WC;
    constexpr int PXB = PK ? 32 : 64, PSH = PK ? 5 : 6;      // bytes of a pixel
    constexpr int PPI = 1024 / PXB;                          // pixels per DMA instruction
    constexpr int LPP = PXB / 16;                            // lanes (16-byte chunks) per pixel
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ RpChan par[KG];                               // (bias folded into the accumulators: par.bias = 0)
    __shared__ RpRes pres[KG];
    __shared__ __attribute__((aligned(16))) int32_t biasl[KG];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = wave % WC, wp = wave / WC;
    const int rho = lane & 31, khalf = lane >> 5;
    const int kbase = blockIdx.y * KG;
    const int chl = wc * 32 + khalf * 16;
    const int ysh = is4(a.y_dt) ? 1 : 0;
    const bool r4 = RES && is4(a.res_dt);
    const RowsWalk walk = rows_walk(blockIdx.x, gridDim.x, g.n_tiles);
    const int step = walk.step, t_end = walk.end;
    int tile = walk.first;

    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, a.N * a.H * a.W * PXB, 0x00020000);
    const int rowb = g.PW * PXB;                             // bytes of an LDS row
    const int ipr = g.PW / PPI;                              // DMA instructions per row
    auto fetch = [&](int t, uint8_t *buf) {
        const int n = t / g.tpi, h0 = (t - n * g.tpi) * g.R;
        const int rows = S2 ? 2 * g.R + 1 : g.R + 2, ih0 = (S2 ? 2 * h0 : h0) - 1;
        const int ni = rows * ipr;
        int row = wave / ipr, at = wave - row * ipr;
        for (int i = wave; i < ni; i += 4) {
            const int j = at * PPI + lane / LPP;             // pixel of the row
            const int iw = S2 ? (j < g.PWh ? 2 * j - 1 : 2 * (j - g.PWh)) : j - 1;
            const int ih = ih0 + row;
            const int px = i * PPI + lane / LPP;
            const int c = (lane & (LPP - 1)) ^ ((PK ? px >> 3 : px >> 2) & (LPP - 1));
            const bool ok = t < t_end && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W && (!S2 || j < 2 * g.PWh);
            const uint32_t off = ok ? (uint32_t)((n * a.H + ih) * a.W + iw) * PXB + c * 16 : 0x80000000u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(buf + i * 1024), 16, (int)off, 0, 0, 0);
            at += 4;
            while (at >= ipr) { at -= ipr; ++row; }
        }
    };
    fetch(tile, lds);
    asm volatile("" ::: "memory");
    // ---- weights: the 18 fragments of channels kbase + 32 wc .. + 31 ----
    v4i wf[18];
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)a.w_f, 0, (a.K / 32) * 9 * 2048, 0x00020000);
        const int o0 = __builtin_amdgcn_readfirstlane((kbase / 32 + wc) * 9 * 2048);
#pragma unroll
        for (int h = 0; h < 18; ++h) wf[h] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, o0 + h * 1024, 0);
    }
    int wide = 0;
    if (tid < KG) {
        const int k = kbase + tid;
        const int32_t b = a.b[k], c = a.c[k];
        RpChan p{0, b, c, 0, 0};
        if (c > 32 || ((int64_t)b >> (c - 1)) != 0) wide = 1;
        else p.bs = (int32_t)((uint32_t)b << (32 - c));
        par[tid] = p;
        biasl[tid] = a.bias[k];
        if (RES) {
            const int32_t rb = a.res_b[k], rc = a.res_c[k];
            if (rc > 31 || rb >= (1 << 22)) wide = 1;
            pres[tid] = RpRes{rb, rc};
        }
    }
    wide = __syncthreads_or(wide);
    int32_t bs[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) bs[i] = par[chl + i].bs;

    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc((void *)a.y, 0, (int)(((int64_t)a.M * a.K) >> ysh), 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_r = __builtin_amdgcn_make_buffer_rsrc((void *)(RES ? a.res : a.x), 0, RES ? (int)(((int64_t)a.M * a.K) >> (r4 ? 1 : 0)) : 0, 0x00020000);
    const int n_px = g.R * a.Q;                              // output pixels of a full tile
    const uint32_t nsh = khalf * 4;
    int32_t lo = a.lo, hi = a.hi;
    asm volatile("" : "+v"(lo), "+v"(hi));
    int64_t half = (int64_t)1 << 31;
    asm volatile("" : "+v"(half));

    // NTP (1 or 2) MFMA column tiles, t0 and t0 + 1, of the tile in `cur` whose first output pixel is m0
    auto compute = [&](auto ntpc, int t0, const uint8_t *cur, int64_t m0, int valid) {
        constexpr int NTP = decltype(ntpc)::value;
        uint32_t base[NTP][S2 ? 2 : 3], yoff[NTP];
        uint32_t resw[NTP][4] = {};
#pragma unroll
        for (int t = 0; t < NTP; ++t) {
            const int i = (t0 + t) * 32 + rho;
            yoff[t] = i < valid ? (uint32_t)((m0 + i) * a.K + kbase + chl) : 0x80000000u;
            if constexpr (RES) {
                if (r4) {
                    const v2i v = __builtin_amdgcn_raw_buffer_load_b64(rs_r, (int)(i < valid ? yoff[t] >> 1 : 0x80000000u), 0, 0);
                    resw[t][0] = (uint32_t)v[0]; resw[t][1] = (uint32_t)v[1];
                } else {
                    const v4i v = __builtin_amdgcn_raw_buffer_load_b128(rs_r, (int)yoff[t], 0, 0);
                    resw[t][0] = (uint32_t)v[0]; resw[t][1] = (uint32_t)v[1]; resw[t][2] = (uint32_t)v[2]; resw[t][3] = (uint32_t)v[3];
                }
            }
            const int ic = i < n_px ? i : n_px - 1;
            const int row = rows_row((uint32_t)ic, g.mq);
            const uint32_t p = (uint32_t)((S2 ? 2 * row : row) * g.PW + (ic - row * a.Q)) << PSH;
            // the three columns of the window (stride 2: even plane at +0 and +1, odd plane PWh pixels on)
#pragma unroll
            for (int s = 0; s < (S2 ? 2 : 3); ++s) {
                const uint32_t v = p + s * PXB;
                base[t][s] = PK ? v + (((v >> 8) & 1) << 4) : v + ((((v >> 8) & 3) ^ khalf) << 4);
            }
        }
        v16i acc[NTP];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v4i bq = *(const v4i *)(biasl + chl + 4 * q);
#pragma unroll
            for (int t = 0; t < NTP; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[t][4 * q + i] = bq[i];
        }
        v4i bf[2][NTP];
        auto frag = [&](auto hc) {
            constexpr int h = decltype(hc)::value, tap = h / 2, r = tap / 3, s = tap % 3;
#pragma unroll
            for (int t = 0; t < NTP; ++t) {
                uint32_t v;
                if constexpr (S2) v = s == 1 ? base[t][0] + (uint32_t)(r * rowb + (g.PWh << PSH)) : base[t][s / 2] + (uint32_t)(r * rowb);
                else v = base[t][s] + (uint32_t)(r * rowb);
                bf[h & 1][t] = *(const v4i *)(cur + (v ^ (PK ? (h & 1) << 4 : (h & 1) << 5)));
            }
        };
        frag(std::integral_constant<int, 0>{});
        static_for<0, 18>([&](auto hc) {
            constexpr int h = decltype(hc)::value;
            if constexpr (h + 1 < 18) frag(std::integral_constant<int, h + 1>{});
#pragma unroll
            for (int t = 0; t < NTP; ++t) {
                v4i b = bf[h & 1][t];
                if constexpr (PK) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) b[e] = (int)(((uint32_t)b[e] >> nsh) & 0x0F0F0F0Fu);
                }
                acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[h], b, acc[t], 0, 0, 0);
            }
        });
        // ---- epilogue ----
        uint32_t out[NTP][4];
        if constexpr (RES) {
            if (r4)
#pragma unroll
                for (int t = 0; t < NTP; ++t) {               // nibbles -> one channel per byte
                    const uint32_t v[2] = {resw[t][0], resw[t][1]};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t n = (v[q >> 1] >> (16 * (q & 1))) & 0xffffu;
                        resw[t][q] = (n & 0xfu) | ((n & 0xf0u) << 4) | ((n & 0xf00u) << 8) | ((n & 0xf000u) << 12);
                    }
                }
        }
        if (wide) {
#pragma unroll
            for (int t = 0; t < NTP; ++t) {
                uint32_t o[2][4];
                const uint32_t rw[2][4] = {{resw[t][0], resw[t][1], resw[t][2], resw[t][3]}, {0, 0, 0, 0}};
                rp_epilogue<1>(acc[t], acc[t], par + chl, pres + chl, RES, a.res_dt == HAWQ_S8, rw, 1, a.lo, a.hi, o);
#pragma unroll
                for (int q = 0; q < 4; ++q) out[t][q] = o[0][q];
            }
        } else {
            int32_t y[NTP][16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                int32_t b = bs[i];
                asm volatile("" : "+v"(b));                   // (keeps the product one 32 x 32 + 64 multiply-add)
#pragma unroll
                for (int t = 0; t < NTP; ++t) y[t][i] = (int32_t)(((int64_t)acc[t][i] * (int64_t)b + half) >> 32);
            }
            if constexpr (RES) {
                auto add = [&](auto sc) {
                    constexpr bool SGN = decltype(sc)::value;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const RpRes p = pres[chl + i];
                        const int32_t rr = (int32_t)(1u << ((p.rc - 1) & 31));
#pragma unroll
                        for (int t = 0; t < NTP; ++t) {
                            const int32_t r = SGN ? __builtin_amdgcn_sbfe((int32_t)resw[t][i >> 2], 8 * (i & 3), 8)
                                                  : (int32_t)__builtin_amdgcn_ubfe(resw[t][i >> 2], 8 * (i & 3), 8);
                            y[t][i] += (__mul24(r, p.rb) + rr) >> p.rc;
                        }
                    }
                };
                if (a.res_dt == HAWQ_S8) add(std::true_type{});
                else add(std::false_type{});
            }
#pragma unroll
            for (int t = 0; t < NTP; ++t) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    int32_t v;
                    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(v) : "v"(y[t][i]), "v"(lo), "v"(hi));
                    y[t][i] = v;
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    out[t][q] = __builtin_amdgcn_perm((uint32_t)y[t][4 * q + 1], (uint32_t)y[t][4 * q], 0x0c0c0400u) |
                                __builtin_amdgcn_perm((uint32_t)y[t][4 * q + 3], (uint32_t)y[t][4 * q + 2], 0x04000c0cu);
            }
        }
#pragma unroll
        for (int t = 0; t < NTP; ++t) {
            if (ysh) {
                auto nib = [](uint32_t d) { return (d & 0xfu) | ((d >> 4) & 0xf0u) | ((d >> 8) & 0xf00u) | ((d >> 12) & 0xf000u); };
                const uint32_t o = yoff[t] & 0x80000000u ? yoff[t] : yoff[t] >> 1;
                __builtin_amdgcn_raw_buffer_store_b64((v2i){(int)(nib(out[t][0]) | (nib(out[t][1]) << 16)), (int)(nib(out[t][2]) | (nib(out[t][3]) << 16))}, rs_y, (int)o, 0, 0);
            } else {
                __builtin_amdgcn_raw_buffer_store_b128((v4i){(int)out[t][0], (int)out[t][1], (int)out[t][2], (int)out[t][3]}, rs_y, (int)yoff[t], 0, 0);
            }
        }
    };

    int cur = 0;
    for (; tile < t_end; tile += step) {
        // (every wave's part of this tile's rows has landed; and nobody reads the other buffer any more)
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (tile + step < t_end) fetch(tile + step, lds + (cur ^ 1) * g.buf);
        const uint8_t *buf = lds + cur * g.buf;
        const int n = tile / g.tpi, h0 = (tile - n * g.tpi) * g.R;
        const int64_t m0 = ((int64_t)n * a.P + h0) * a.Q;
        const int rows = a.P - h0 < g.R ? a.P - h0 : g.R, valid = rows * a.Q, nt = (valid + 31) >> 5;
        // this wave's column tiles: the first or second half (of five: three and two, not two pairs and a single)
        const int half = (nt + 1) >> 1, t0 = WP == 1 || wp == 0 ? 0 : half, t1 = WP == 1 || wp == 1 ? nt : half;
        for (int t = t0; t < t1; t += 2) {
            if (t + 1 < t1) compute(std::integral_constant<int, 2>{}, t, buf, m0, valid);
            else compute(std::integral_constant<int, 1>{}, t, buf, m0, valid);
        }
        cur ^= 1;
    }
}

// ---- host side ----

static bool rows_plan(const ConvArgs &a, RowsArgs &g) {
    return rows_plan(a.N, a.W, a.P, a.Q, a.stride_h == 2, is4(a.x_dt), g);
}

// Where this form is preferred, against the kernel that takes the layer otherwise (conv3x3_c64.hip for 64 -> 64 at stride 1 and
// up to 62 columns, else the tiled kernel), swept over images of 20x20 to 112x112 and 9000 to 400000 output pixels.  Either
// kernel's time climbs in steps, a round of workgroups each, so no line by pixels alone holds for every image size (with one,
// from 50000 pixels and for stride 2 from 12000 on, layers were up to 1.7 times slower than before: 28x28 at batch 66 7.4 us ->
// 12.5).  The estimates of rows_faster place the steps:
//   stride 1, 64 -> 64, up to 62 columns, with a shortcut: 56x56 at batch 17 8.7 us against 9.2, 19 10.3 against 9.4 (left), 64 18.4
//   against 22.1, 128 27.2 against 35.9; without: 32 9.8 against 10.7, 40 12.5 against 11.2 (left), 64 15.6 against 15.1 alone,
//   but inside the networks ahead (ResNet50 at batch 128 as 64 + 64 1077 us with it, 1085 without), 128 24.1 against 25.6;
//   stride 2, 56x56 64 -> 128: batch 32 8.3 against 8.8, 48 10.4 against 11.7, 128 16.0 against 21.0; packed, 64 12.2 against 14.0, 66
//   14.2 against 12.8 (left).
//   stride 1, 64 -> 128: 112x112 batch 4 9.7 against 11.5, 56x56 19 16.5 against 14.0 (left), 96 33.7 against 48.2.
// More columns at 64 channels (112x112: 7.2 us against 8.6 at batch 4, 24.0 against 45.0 at 32; packed 7.8 against 10.5 at 4) come here
// from 50000 pixels on.  Packed operands cost eight vector operations per fragment here: up to 62 columns stride 1 stays with
// conv3x3_c64 (14.7 against 17.9 us at batch 64).  Fewer pixels: the split-reduction forms.
// (Measured and dropped: three workgroups per compute unit -- the registers allow two; reading fragments two or three
// half-steps ahead with a fixed schedule; requantising a pair of column tiles between the next pair's MFMAs.  What a tile costs
// beside its MFMAs -- the matrix pipe is busy 0.20 to 0.36 of the time -- is its start-up (3 us), the fetch's issue (0.7 us), the bank
// conflicts at row ends and the epilogue, which nothing overlaps within a wave.)

// Microseconds of this kernel and of the other one, fitted to 2400 layers of 64 to 512 output channels (each row 2 to 5 % rms).  Here:
// rounds of 256 workgroups, times the column tiles of a wave and the KB of a tile's rows, and the MB that move; there: rounds of
// workgroups, and the MB.  `margin`: how far below the other estimate this one has to be (64 -> 64 without a shortcut may be 3 %
// above it: inside a network, with its input still in cache, it gains that: ResNet18 at batch 26 208 us without, 203 with it).
// Beside another stream's kernels (corun) the end of a round idles nothing, and this kernel's fewer bytes per output decide: ResNet18 at
// batch 103 as 56 + 47 354 us by the estimates, 338 with it throughout; at 206 514 and 493; ResNet50 at 96 894 and 879.
struct RowsCost { double start, tile, kb, mb, o_start, o_round, o_mb, margin; };

static bool rows_faster(const ConvArgs &a, const RowsArgs &g, int wc, int ncg) {
    const bool s2 = a.stride_h == 2, four = is4(a.x_dt), res = a.res != nullptr;
    const RowsCost c = !s2 && a.K == 64 ? (res ? RowsCost{5.23, 0.491, 0.0, 0.123, 4.67, 2.363, 0.0, a.M > 65536 ? 1.0 : 0.94}     // conv3x3_c64
                                               : RowsCost{4.66, 0.351, 0.005, 0.168, 4.6, 1.255, 0.067, a.M > 65536 ? 1.03 : 1.0})
                     : !s2              ? (res ? RowsCost{6.09, 0.51, 0.016, 0.08, 4.55, 3.35, 0.163, 1.0} : RowsCost{5.08, 0.51, 0.012, 0.075, 3.64, 3.2, 0.198, 1.0})
                     : four             ? (a.K == 64 ? RowsCost{5.33, 0.57, 0.008, 0.103, 3.43, 4.0, 0.394, 1.0} : RowsCost{5.22, 0.74, 0.008, 0.035, 4.57, 4.13, 0.154, 1.0})
                     : a.K == 64        ? RowsCost{4.75, 0.41, 0.015, 0.052, 3.0, 3.93, 0.172, 0.97}
                     : wc == 4          ? RowsCost{4.99, 0.553, 0.02, 0.013, 3.66, 3.74, 0.083, 0.97}
                                        : RowsCost{4.65, 0.505, 0.024, 0.0, 3.89, 2.84, 0.196, 0.97};
    const int64_t px_tiles = ((int64_t)a.M + 127) / 128;      // 256 of them are a round of conv3x3_c64, 512 one of the tiled kernel's 64 x 128 tiles
    const int64_t o_rounds = a.K != 64 ? (px_tiles * ((a.K + 127) / 128) + 255) / 256 : s2 ? (px_tiles + 511) / 512 : (px_tiles + 255) / 256;
    const double rounds = (double)(((int64_t)g.n_tiles * ncg + 255) / 256), tiles = wc == 4 ? g.nt : (g.nt + 1) / 2;
    const double mb = 1e-6 / (four ? 2 : 1) * a.M * (64 * a.stride_h * a.stride_w + a.K * (res ? 2 : 1));
    return c.start + rounds * (c.tile * tiles + c.kb / 1024 * g.buf) + c.mb * mb < c.margin * (c.o_start + c.o_round * (double)o_rounds + c.o_mb * mb);
}

bool conv3x3_rows_eligible(const ConvArgs &a, int x_hi) {
    if (a.R != 3 || a.S != 3 || a.C != 64 || a.pad_h != 1 || a.pad_w != 1 || a.stride_h != a.stride_w || (a.stride_h != 1 && a.stride_h != 2)) return false;
    const bool s2 = a.stride_h == 2, four = is4(a.x_dt), wide_image = !s2 && a.W > 62 && (a.K == 64 || four);
    if (a.M < (s2 && !four ? 12000 : 50000) || (!s2 && four && !wide_image)) return false;
    if (a.w_f == nullptr || a.b == nullptr || a.xs != nullptr || a.K % 64 != 0) return false;
    if (a.x_dt == HAWQ_U4) { if (a.w_dt != HAWQ_S4) return false; }
    else if (a.w_dt != HAWQ_S8 || (a.x_dt == HAWQ_U8 ? x_hi > 127 : a.x_dt != HAWQ_S8)) return false;
    if (a.y_dt != HAWQ_U8 && a.y_dt != HAWQ_S8 && a.y_dt != HAWQ_U4) return false;
    if (a.res != nullptr && a.res_dt != HAWQ_U8 && a.res_dt != HAWQ_S8 && a.res_dt != HAWQ_U4) return false;
    if (((uintptr_t)a.x | (uintptr_t)a.y | (uintptr_t)a.res) & 15) return false;
    if (!rows_offsets_fit(a.M, a.K)) return false;
    RowsArgs g{};
    int wc = 0, ncg = 0, gx = 0;
    if (!rows_plan(a, g) || !rows_grid(a.K, g.n_tiles, wc, ncg, gx)) return false;
    return wide_image || a.corun || rows_faster(a, g, wc, ncg);
}

hawq_status launch_conv3x3_rows(const ConvArgs &a, hipStream_t s) {
    RowsArgs g{};
    int wc = 0, ncg = 0, gx = 0;
    if (!rows_plan(a, g) || !rows_grid(a.K, g.n_tiles, wc, ncg, gx)) return HAWQ_ERR_UNSUPPORTED;
    const bool s2 = a.stride_h == 2, pk = is4(a.x_dt), res = a.res != nullptr;
    const dim3 grid(gx, ncg);
    const size_t lds = 2 * (size_t)g.buf;
    auto go = [&](auto wcc, auto s2c, auto pkc, auto rc) {
        conv3x3_rows_kernel<decltype(wcc)::value, decltype(s2c)::value, decltype(pkc)::value, decltype(rc)::value><<<grid, 256, lds, s>>>(a, g);
    };
    auto on_r = [&](auto wcc, auto s2c, auto pkc) { if (res) go(wcc, s2c, pkc, std::true_type{}); else go(wcc, s2c, pkc, std::false_type{}); };
    auto on_p = [&](auto wcc, auto s2c) { if (pk) on_r(wcc, s2c, std::true_type{}); else on_r(wcc, s2c, std::false_type{}); };
    auto on_s = [&](auto wcc) { if (s2) on_p(wcc, std::true_type{}); else on_p(wcc, std::false_type{}); };
    if (wc == 4) on_s(std::integral_constant<int, 4>{}); else on_s(std::integral_constant<int, 2>{});
    return check_launch();
}

}  // namespace hawq
