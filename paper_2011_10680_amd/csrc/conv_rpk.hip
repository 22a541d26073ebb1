// 3x3 / stride 1 / pad 1 convolution with the pixel operand resident in LDS and the reduction split over the waves: the
// form of conv_rp.hip for launches that do not fill the chip with its tiles.
//
// conv_rp's workgroup gives every wave 32 output channels and the whole reduction; with few pixel tiles most compute units
// then idle while each busy one streams all the weights of 128 or 256 channels.  Here a workgroup owns only 32 (64) channels
// of a tile, and its WK waves divide the *input channels* among themselves: a wave multiplies its slice of every tap, so it
// needs 9 or 18 weight fragments in all -- every one of them is requested up front, next to the patch -- and its K loop is
// that many half-steps, without a barrier.  The partial tiles meet in LDS, where the patch was.
//   * Patch: the run of BP + 2W + 2 input pixels under the tile (see conv_rp.hip), fetched by LDS-DMA.  A DMA instruction
//     fills 1 KB of consecutive LDS, so rows are not padded; instead the 16-byte chunks of a row are permuted (chunk ^ row)
//     on the source side, which puts the sixteen rows of a 128-bit LDS access into sixteen different banks.  Taps outside
//     the image read a row of zeros.  LDS is sized at launch from the image width.
//   * PK (packed 4-bit): the patch stays packed; a lane takes the low or the high nibbles of its chunk on the way into the
//     MFMA, the order in which the fragment copy expanded the weights.
// What bounds it: operand delivery -- a compute unit draws about 57 KB/us from behind its L2, and a 32-channel tile needs
// (9 C 32 + patch) bytes -- and then launch and drain.
#include "rp.h"

namespace hawq {

template <int CCH, int TP, int WC, int WK, bool PK>
__global__ void __launch_bounds__(64 * WC * WK) conv_rpk_kernel(const RpArgs a) {
    constexpr int T = 64 * WC * WK;
    constexpr int BP = 32 * TP;                       // output pixels of the tile
    constexpr int C = 64 * CCH, CB = PK ? C / 2 : C;  // channels, bytes of a patch row
    constexpr int NC = CB / 16;                       // 16-byte chunks of a row
    constexpr int RSH = CB >= 256 ? 0 : CB == 128 ? 1 : CB == 64 ? 2 : 3;   // rows per 256 bytes (log2)
    constexpr int XM = NC < 16 ? NC - 1 : 15;         // chunk permutation: chunk ^ ((row >> RSH) & XM)
    constexpr int HPT = 2 * CCH / WK;                 // half-steps (32 input channels) of a tap per wave
    constexpr int NH = 9 * HPT;
    constexpr int R = WK >= 8 ? 4 : (WC * WK >= 8 ? 2 : WK);   // partial tiles per channel group after the first exchange
    static_assert(HPT >= 1 && NH <= 18 && WK / R <= 2, "split");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ RpChan par[32 * WC];
    __shared__ RpRes pres[32 * WC];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wc = wave / WK;
    const int rho = lane & 31, khalf = lane >> 5;
    const int W = a.W;
    const int ncg = a.K1 / (32 * WC);
    // channel groups vary fastest: workgroup b runs on XCD b % 8, so an XCD's L2 keeps an eighth of the weights
    const int cg = (int)(blockIdx.x % (uint32_t)ncg), m0 = (int)(blockIdx.x / (uint32_t)ncg) * BP;
    const int kbase = cg * 32 * WC;

    // ---- patch rows 0 .. BP + 2W + 1 = flat pixels m0 - W - 1 ..., then a row of zeros, by LDS-DMA ----
    const int rows = BP + 2 * W + 2;                  // (row `rows` and what the last instruction covers beyond it: zeros)
    {
        constexpr int RPI = 1024 / CB > 0 ? 1024 / CB : 1;   // rows per instruction
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, (int)((int64_t)a.M * CB), 0x00020000);
        const int ninst = (rows + 1 + RPI - 1) / RPI;
        const int r_in = lane / NC, pos = lane % NC;
        for (int i = wave; i < ninst; i += WC * WK) {
            const int row = i * RPI + r_in;
            const int px = m0 - W - 1 + row;
            const uint32_t off = (px >= 0 && row < rows) ? (uint32_t)px * CB + ((pos ^ ((row >> RSH) & XM)) << 4) : 0x80000000u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + i * 1024), 16, (int)off, 0, 0, 0);
        }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    // ---- the wave's weight fragments, all of them ----
    v4i af[NH];
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)a.w1f, 0, (a.K1 / 32) * 9 * CCH * 2048, 0x00020000);
        const int o0 = __builtin_amdgcn_readfirstlane(((kbase / 32 + wc) * 9 * CCH * 2 + wk * HPT) * 1024);
#pragma unroll
        for (int h = 0; h < NH; ++h) af[h] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, o0 + ((h / HPT) * 2 * CCH + h % HPT) * 1024, 0);
    }
    // ---- parameters, and the shortcut bytes of the tiles this wave will finish ----
    const bool has_res = a.res != nullptr;
    const int ysh = a.y4 ? 1 : 0;                     // a packed 4-bit output holds two channels per byte
    constexpr int NF = (TP + R - 1) / R;              // tiles a wave finishes (waves wk < R)
    uint32_t resw[NF][4] = {}, yoff[NF];
    const int chl = wc * 32 + khalf * 16;
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)(has_res ? a.res : a.x), 0, has_res ? (int)((int64_t)a.M * a.K1) : 0, 0x00020000);
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int t = wk + j * R;
            const int64_t m = (int64_t)m0 + t * 32 + rho;
            const bool ok = wk < R && t < TP && m < a.M;
            yoff[j] = ok ? (uint32_t)((m * a.K1 + kbase + chl) >> ysh) : 0x80000000u;
            if (has_res) {
                const v4i v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)yoff[j], 0, 0);
                resw[j][0] = (uint32_t)v[0]; resw[j][1] = (uint32_t)v[1]; resw[j][2] = (uint32_t)v[2]; resw[j][3] = (uint32_t)v[3];
            }
        }
    }
    int wide = 0;
    if (tid < 32 * WC) {
        const int k = kbase + tid;
        const int32_t b = a.b1[k], c = a.c1[k], bias = a.bias1[k];
        RpChan p{0, b, c, bias, 0};
        if (c > 32 || ((int64_t)b >> (c - 1)) != 0) wide = 1;
        else {
            p.bs = (int32_t)((uint32_t)b << (32 - c));
            p.Rs = (int64_t)((uint64_t)((int64_t)bias * (int64_t)b + ((int64_t)1 << (c - 1))) << (32 - c));
        }
        par[tid] = p;
        if (has_res) {
            const int32_t rb = a.res_b[k], rc = a.res_c[k];
            if (rc > 31 || rb >= (1 << 22)) wide = 1;
            pres[tid] = RpRes{rb, rc};
        }
    }
    // ---- which taps of the lane's pixels lie inside the image ----
    uint32_t vmask[TP];
    {
        const int H = a.H, HW = H * W;
#pragma unroll
        for (int tp = 0; tp < TP; ++tp) {
            const int64_t m = (int64_t)m0 + tp * 32 + rho;
            const bool pv = m < a.M;
            const int rem = pv ? (int)((uint32_t)m % (uint32_t)HW) : 0;
            const int yy = rem / W, xx = rem - yy * W;
            uint32_t mask = 0;
#pragma unroll
            for (int r = 0; r < 3; ++r)
#pragma unroll
                for (int s = 0; s < 3; ++s)
                    if (pv && (unsigned)(yy + r - 1) < (unsigned)H && (unsigned)(xx + s - 1) < (unsigned)W) mask |= 1u << (r * 3 + s);
            vmask[tp] = mask;
        }
    }
    wide = __syncthreads_or(wide);

    // ---- K loop: 9 HPT half-steps of TP MFMAs; the next half-step's fragments are read while this one is multiplied ----
    v16i acc[TP];
#pragma unroll
    for (int tp = 0; tp < TP; ++tp)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[tp][i] = 0;
    v4i bf[2][TP];
    uint32_t sel[TP];
    const uint32_t nsh = khalf * 4;                   // PK: the nibble this lane half takes
    // 16-byte chunk of half-step q of the wave: two chunks per half-step (one per lane half), or, packed, one shared chunk
    auto fetch = [&](auto hc, auto bc) {
        constexpr int h = decltype(hc)::value, buf = decltype(bc)::value;
        constexpr int tap = h / HPT, j = h % HPT, r = tap / 3, s = tap % 3;
        if constexpr (j == 0) {
            const int shift = r * W + s;
#pragma unroll
            for (int tp = 0; tp < TP; ++tp) {
                const int row = ((vmask[tp] >> tap) & 1u) ? tp * 32 + rho + shift : rows;
                sel[tp] = (uint32_t)row * CB + (((row >> RSH) & XM) << 4);
            }
        }
        const uint32_t c = PK ? (uint32_t)(wk * HPT + j) : (uint32_t)((wk * HPT + j) * 2 + khalf);
#pragma unroll
        for (int tp = 0; tp < TP; ++tp) bf[buf][tp] = *(const v4i *)(lds + (sel[tp] ^ (c << 4)));
    };
    fetch(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
    static_for<0, NH>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        if constexpr (h + 1 < NH) fetch(std::integral_constant<int, h + 1>{}, std::integral_constant<int, (h + 1) % 2>{});
#pragma unroll
        for (int tp = 0; tp < TP; ++tp) {
            v4i b = bf[h % 2][tp];
            if constexpr (PK) {
#pragma unroll
                for (int e = 0; e < 4; ++e) b[e] = (int)(((uint32_t)b[e] >> nsh) & 0x0F0F0F0Fu);
            }
            acc[tp] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[h], b, acc[tp], 0, 0, 0);
        }
    });

    // ---- the partial tiles meet where the patch was ----
    v16i fin[NF];
    rpk_reduce<TP, WC, WK, R, NF>(lds, lane, wk, wc, acc, fin);
    if (wk >= R || wk >= TP) return;
    const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc((void *)a.y, 0, (int)(((int64_t)a.M * a.K1) >> ysh), 0x00020000);
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        if (wk + j * R >= TP) break;
        rpk_store(fin[j], par + chl, pres + chl, has_res, a.res_dt == HAWQ_S8, resw[j], wide, a.lo1, a.hi1, ysh != 0, rsrc_y, yoff[j]);
    }
}

template <int CCH, int TP, int WC, int WK>
static hawq_status rpk_launch(const RpArgs &a, hipStream_t s) {
    constexpr int R = WK >= 8 ? 4 : (WC * WK >= 8 ? 2 : WK);
    const int cb = a.pk ? 32 * CCH : 64 * CCH, bp = 32 * TP;
    const uint32_t nb = (uint32_t)((a.M + bp - 1) / bp) * (uint32_t)(a.K1 / (32 * WC));
    size_t lds = ((size_t)(bp + 2 * a.W + 3) * cb + 1023) / 1024 * 1024;
    const size_t red = (size_t)WC * R * TP * 4096;
    if (red > lds) lds = red;
    if (a.pk) conv_rpk_kernel<CCH, TP, WC, WK, true><<<nb, 64 * WC * WK, lds, s>>>(a);
    else conv_rpk_kernel<CCH, TP, WC, WK, false><<<nb, 64 * WC * WK, lds, s>>>(a);
    return check_launch();
}

// Where this form is preferred (single layers at batch 1 .. 128, weights not in L2; this kernel against the split-reduction
// and the resident-pixel / tiled one): a 64-pixel x 32-channel tile while that is at most one round of workgroups (256
// compute units), 64 x 64 beyond, as long as two workgroups per compute unit hold the launch (C = 256: one -- four waves
// share a reduction there, and conv_rp's half-width tiles take over).
//   7x7 512: batch 4 6.1 us (7.1), 8 6.3 (8.5), 16 6.7 (12.4), 32 9.8 (15.0), 64 16.7 (15.1)
//   14x14 256: batch 4 5.5 (6.3), 8 5.9 (8.6), 16 7.1 (9.5), 32 9.9 (9.5)
//   28x28 128: batch 2 4.5 (4.9), 4 4.7 (6.4), 8 5.7 (8.6), 16 7.6 (10.2), 32 12.3 (10.7)
//   56x56 64: batch 4 4.6 (6.8), 8 5.7 (7.3), 16 7.6 (6.8)
// Below the lower line the split-reduction kernel's smaller tiles put more compute units to work; it moves packed 4-bit
// operands at half the bytes, so its line lies higher there (7x7 512 packed: batch 8 7.1 us here, 6.2 there; 16 7.3, 8.4).
static int rpk_variant(const RpArgs &a) {
    const int cch = a.C / 64;
    if (a.C % 64 != 0 || (cch != 1 && cch != 2 && cch != 4 && cch != 8) || a.K1 % 64 != 0 || a.M <= 0) return 0;
    if (a.res != nullptr && (a.pk || a.y4)) return 0;
    if (((int64_t)(64 + 2 * a.W + 3) * a.C) > (96 << 10)) return 0;    // the patch: LDS
    const int64_t out = (int64_t)a.M * a.K1;
    if (out <= (a.pk || cch == 1 ? 1 << 18 : 3 << 15)) return 0;
    const int64_t narrow = ((int64_t)a.M + 63) / 64 * (a.K1 / 32), wide = narrow / 2;
    switch (cch) {
    case 1: return wide <= 512 ? 1 : 0;
    case 2: return narrow <= 256 ? 2 : wide <= 512 ? 3 : 0;
    case 4: return narrow <= 256 ? 4 : wide <= 256 ? 5 : 0;
    default: return narrow <= 512 ? 6 : 0;
    }
}

bool conv_rpk_shape_ok(const RpArgs &a) { return rpk_variant(a) != 0; }

hawq_status launch_conv_rpk(const RpArgs &a, hipStream_t s) {
    switch (rpk_variant(a)) {
    case 1: return rpk_launch<1, 2, 2, 2>(a, s);
    case 2: return rpk_launch<2, 2, 1, 4>(a, s);
    case 3: return rpk_launch<2, 2, 2, 4>(a, s);
    case 4: return rpk_launch<4, 2, 1, 8>(a, s);
    case 5: return rpk_launch<4, 2, 2, 4>(a, s);
    case 6: return rpk_launch<8, 2, 1, 8>(a, s);
    default: return HAWQ_ERR_UNSUPPORTED;
    }
}

}  // namespace hawq
