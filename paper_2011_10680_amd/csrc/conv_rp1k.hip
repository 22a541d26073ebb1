// 1x1 convolution (any stride) with the pixel operand resident in LDS and the reduction split over the waves: the pointwise
// twin of conv_rpk.hip, for launches that do not fill the chip with the streaming or resident-pixel kernels' tiles.
//
// A workgroup owns a tile of 32 TP pixels x 32 WC channels; its pixels, every channel of them, come to LDS once by LDS-DMA
// (whole rows of C bytes; the 16-byte chunks of a row are permuted on the source side, see conv_rpk.hip), its weights as
// fragments straight into registers, all requested up front, each read by exactly one wave.  WK waves per channel group
// divide the input channels; the partial tiles meet in LDS, where the pixels were.
#include "rp.h"

namespace hawq {

template <int CCH, int TP, int WC, int WK, bool PK>
__global__ void __launch_bounds__(64 * WC * WK) conv_rp1k_kernel(const ConvArgs a) {
    constexpr int BP = 32 * TP;
    constexpr int C = 64 * CCH, CB = PK ? C / 2 : C;
    constexpr int NC = CB / 16;
    constexpr int RSH = CB >= 256 ? 0 : CB == 128 ? 1 : CB == 64 ? 2 : 3;
    constexpr int XM = NC < 16 ? NC - 1 : 15;
    constexpr int NH = 2 * CCH / WK;                  // half-steps (32 input channels) per wave
    constexpr int R = WK >= 8 ? 4 : (WK == 4 && WC >= 2 ? 2 : WK);
    static_assert(NH >= 1 && NH <= 16 && WK / R <= 2, "split");
    extern __shared__ __attribute__((aligned(1024))) uint8_t lds[];
    __shared__ RpChan par[32 * WC];
    __shared__ RpRes pres[32 * WC];

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wc = wave / WK;
    const int rho = lane & 31, khalf = lane >> 5;
    const int ncg = a.K / (32 * WC);
    const int cg = (int)(blockIdx.x % (uint32_t)ncg), m0 = (int)(blockIdx.x / (uint32_t)ncg) * BP;
    const int kbase = cg * 32 * WC;

    // ---- the tile's pixels ----
    {
        constexpr int RPI = CB >= 1024 ? 1 : 1024 / CB, IPR = CB > 1024 ? CB / 1024 : 1;   // rows per DMA instruction, instructions per row
        constexpr int NI = BP / RPI * IPR;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, (int)((int64_t)a.N * a.H * a.W * CB), 0x00020000);
        const bool strided = (a.stride_h | a.stride_w) != 1;
        for (int i = wave; i < NI; i += WC * WK) {
            const int row = IPR > 1 ? i / IPR : i * RPI + lane / NC;
            const int pos = IPR > 1 ? (i % IPR) * 64 + lane : lane % NC;
            const int m = m0 + row;
            int px = m;
            if (strided) {
                const int PQ = a.P * a.Q, n = m / PQ, pq = m - n * PQ, p = pq / a.Q, q = pq - p * a.Q;
                px = (n * a.H + p * a.stride_h) * a.W + q * a.stride_w;
            }
            const uint32_t off = m < a.M ? (uint32_t)px * CB + ((pos ^ ((row >> RSH) & XM)) << 4) : 0x80000000u;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(lds + i * 1024), 16, (int)off, 0, 0, 0);
        }
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    v4i af[NH];
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)a.w_f, 0, ((a.K + 31) / 32) * CCH * 2048, 0x00020000);
        const int o0 = __builtin_amdgcn_readfirstlane(((kbase / 32 + wc) * CCH * 2 + wk * NH) * 1024);
#pragma unroll
        for (int h = 0; h < NH; ++h) af[h] = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, o0 + h * 1024, 0);
    }
    // ---- parameters, and the shortcut bytes of the tiles this wave will finish ----
    const bool has_res = a.res != nullptr, r4 = is4(a.res_dt);
    const int ysh = is4(a.y_dt) ? 1 : 0;
    constexpr int NF = (TP + R - 1) / R;
    uint32_t resw[NF][4] = {}, yoff[NF];
    const int chl = wc * 32 + khalf * 16;
    {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)(has_res ? a.res : a.x), 0, has_res ? (int)(((int64_t)a.M * a.K) >> (r4 ? 1 : 0)) : 0, 0x00020000);
#pragma unroll
        for (int j = 0; j < NF; ++j) {
            const int t = wk + j * R;
            const int64_t m = (int64_t)m0 + t * 32 + rho;
            const bool ok = wk < R && t < TP && m < a.M;
            const uint32_t e = (uint32_t)(m * a.K + kbase + chl);
            yoff[j] = ok ? e >> ysh : 0x80000000u;
            if (has_res && r4) {      // eight bytes of nibbles -> one channel per byte
                const v2i v = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)(ok ? e >> 1 : 0x80000000u), 0, 0);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t n = ((uint32_t)v[q >> 1] >> (16 * (q & 1))) & 0xffffu;
                    resw[j][q] = (n & 0xfu) | ((n & 0xf0u) << 4) | ((n & 0xf00u) << 8) | ((n & 0xf000u) << 12);
                }
            } else if (has_res) {
                const v4i v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(ok ? e : 0x80000000u), 0, 0);
                resw[j][0] = (uint32_t)v[0]; resw[j][1] = (uint32_t)v[1]; resw[j][2] = (uint32_t)v[2]; resw[j][3] = (uint32_t)v[3];
            }
        }
    }
    int wide = 0;
    if (tid < 32 * WC) {
        const int k = kbase + tid;
        const int32_t b = a.b[k], c = a.c[k], bias = a.bias[k];
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
    wide = __syncthreads_or(wide);

    v16i acc[TP];
#pragma unroll
    for (int tp = 0; tp < TP; ++tp)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[tp][i] = 0;
    v4i bf[2][TP];
    uint32_t sel[TP];
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) {
        const int row = tp * 32 + rho;
        sel[tp] = (uint32_t)row * CB + (((row >> RSH) & XM) << 4);
    }
    const uint32_t nsh = khalf * 4;                   // PK: the nibble this lane half takes
    auto fetch = [&](auto hc, auto bc) {
        constexpr int h = decltype(hc)::value, buf = decltype(bc)::value;
        const uint32_t c = PK ? (uint32_t)(wk * NH + h) : (uint32_t)((wk * NH + h) * 2 + khalf);
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
    v16i fin[NF];
    rpk_reduce<TP, WC, WK, R, NF>(lds, lane, wk, wc, acc, fin);
    if (wk >= R || wk >= TP) return;
    const __amdgpu_buffer_rsrc_t rsrc_y = __builtin_amdgcn_make_buffer_rsrc((void *)a.y, 0, (int)(((int64_t)a.M * a.K) >> ysh), 0x00020000);
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        if (wk + j * R >= TP) break;
        rpk_store(fin[j], par + chl, pres + chl, has_res, a.res_dt == HAWQ_S8, resw[j], wide, a.lo, a.hi, ysh != 0, rsrc_y, yoff[j]);
    }
}

template <int CCH, int TP, int WC, int WK>
static hawq_status rp1k_launch(const ConvArgs &a, hipStream_t s) {
    constexpr int R = WK >= 8 ? 4 : (WK == 4 && WC >= 2 ? 2 : WK);
    const bool pk = is4(a.x_dt);
    const int bp = 32 * TP;
    const uint32_t nb = (uint32_t)((a.M + bp - 1) / bp) * (uint32_t)(a.K / (32 * WC));
    size_t lds = (size_t)bp * (pk ? 32 * CCH : 64 * CCH);
    const size_t red = (size_t)WC * R * TP * 4096;
    if (red > lds) lds = red;
    if (lds < 1024) lds = 1024;
    if (pk) conv_rp1k_kernel<CCH, TP, WC, WK, true><<<nb, 64 * WC * WK, lds, s>>>(a);
    else conv_rp1k_kernel<CCH, TP, WC, WK, false><<<nb, 64 * WC * WK, lds, s>>>(a);
    return check_launch();
}

// Where this form is preferred.  Between about 2^18 outputs (below, the split-reduction kernel's smaller tiles win; it moves
// packed operands at half the bytes, so its line lies at 2^19 there, and long reductions come here earlier) and the point
// where the launch is more than one or two workgroups per compute unit (beyond, the streaming, resident-pixel and tiled
// kernels win: they amortise a workgroup's start-up).  Measured per layer, weights not in L2, this kernel (the one it replaces):
//   1024 -> 256 at 14x14: batch 8 5.0 us (6.3), 16 6.4 (9.3), 32 8.8 (9.5), 64 15.0 (11.8)
//   2048 -> 512 at 7x7: batch 4 4.9 (5.4), 8 5.2 (6.0), 16 6.5 (8.2), 32 11.3 (9.5)
//   512 -> 2048 + shortcut at 7x7: batch 8 5.3 (9.0), 16 6.0 (9.4), 32 8.5 (9.9), 64 13.7 (10.7)
//   1024 -> 512 / 2: batch 16 5.0 (6.2), 32 6.5 (8.1); 512 -> 128 at 28x28: batch 8 4.9 (6.3), 16 5.6 (6.6), 32 8.7 (8.8)
//   256 -> 1024 + shortcut at 14x14: batch 4 4.7 (5.5), 8 5.6 (6.7), 16 7.5 (7.2); 128 -> 512 + shortcut: batch 4 5.0 (6.4), 8 6.7 (6.8)
//   256 -> 128 / 2: batch 8 4.5 (5.4), 16 4.9 (6.1), 32 6.5 (7.5), 64 11.1 (10.3); 256 -> 64: batch 4 4.2 (4.6), 8 5.2 (6.1), 32 11.7 (11.4)
// The variant: tiles of 64 channels (32 at C = 2048) and 64 pixels (32 from C = 1024 on) while they are at most one
// workgroup per compute unit, the next larger tile beyond -- that one as far as it is the faster, which depends on what takes the
// layer otherwise.  In workgroups of 64 x 64, against the kernel that takes over:
//   C = 256, no shortcut, 8-bit, K >= 256: to 512 (256 -> 512: 0.92 of the tiled kernel's time at 384, 1.02 at 512, 1.19 at 600; one round
//     of its tiles reaches to 1024).  Packed or K = 128: to 1024 (0.89 to 1.0).  K not a multiple of 128: 64 x 64 to 256 (192 channels:
//     1.07 to 1.12 beyond), packed or K = 64 to 512 (0.79 to 0.93, 0.82 to 0.92).
//   C = 512: to 512 (packed 1.13 to 1.23 at 600 to 704, 8-bit with K = 128 or stride 2 1.04 to 1.11) -- to 800 where the resident-pixel
//     kernel would take the layer, which is no faster there (0.88 to 1.01).
//   C = 1024: to 256 against the tiled kernel (1.0 to 1.10 beyond), to 400 against the resident-pixel one (0.75 to 0.95).
//   C = 128, packed, no shortcut: below the streaming kernel's 8192 pixels (1.03 beyond).
static int rp1k_variant(const ConvArgs &a) {
    if (a.K % 64 != 0 || a.M <= 0) return 0;
    const int64_t out = (int64_t)a.M * a.K;
    const bool pk = is4(a.x_dt), res = a.res != nullptr, k128 = a.K % 128 == 0;
    if (out <= (pk ? 1 << 19 : a.C >= 2048 ? 3 << 15 : a.C >= 1024 ? 1 << 17 : 1 << 18)) return 0;
    const int64_t t64 = ((int64_t)a.M + 63) / 64, t32 = ((int64_t)a.M + 31) / 32, g = a.K / 64;
    // (the layer is conv_rp1.hip's otherwise: see make_rp1_args)
    const bool rp1 = !pk && a.K % 256 == 0 && a.stride_h == 1 && a.stride_w == 1 && !is4(a.y_dt) && !(res && is4(a.res_dt));
    switch (a.C) {
    case 128: return k128 && t64 * (g / 2) <= 256 && !(pk && !res && a.M >= 8192) ? 1 : 0;
    case 256:
        if (t64 * g <= (!k128 && !res && (pk || a.K == 64) ? 512 : 256)) return 2;
        return k128 && t64 * (g / 2) <= (!res && (pk || a.K == 128 || a.K >= 2048) ? 512 : 256) ? 3 : 0;
    case 512: return t64 * g <= 256 ? 4 : k128 && t64 * (g / 2) <= (rp1 ? 400 : 256) ? 5 : 0;
    case 1024: return t32 * g <= 256 ? 6 : t64 * g <= (rp1 ? 400 : 256) ? 7 : 0;
    case 2048: return t32 * (2 * g) <= 256 ? 8 : t64 * (2 * g) <= 256 ? 9 : 0;
    default: return 0;
    }
}

bool conv_rp1k_eligible(const ConvArgs &a, int x_hi) {
    if (a.R != 1 || a.S != 1 || a.pad_h != 0 || a.pad_w != 0 || a.w_f == nullptr || a.b == nullptr || a.xs != nullptr) return false;
    if (a.x_dt == HAWQ_U4) { if (a.w_dt != HAWQ_S4) return false; }
    else if (a.w_dt != HAWQ_S8 || (a.x_dt == HAWQ_U8 ? x_hi > 127 : a.x_dt != HAWQ_S8)) return false;
    if (a.y_dt != HAWQ_U8 && a.y_dt != HAWQ_S8 && a.y_dt != HAWQ_U4) return false;
    if (a.res != nullptr && a.res_dt != HAWQ_U8 && a.res_dt != HAWQ_S8 && a.res_dt != HAWQ_U4) return false;
    if (((uintptr_t)a.x | (uintptr_t)a.y | (uintptr_t)a.res) & 15) return false;
    return rp1k_variant(a) != 0;
}

hawq_status launch_conv_rp1k(const ConvArgs &a, hipStream_t s) {
    switch (rp1k_variant(a)) {
    case 1: return rp1k_launch<2, 2, 4, 2>(a, s);
    case 2: return rp1k_launch<4, 2, 2, 2>(a, s);
    case 3: return rp1k_launch<4, 2, 4, 2>(a, s);
    case 4: return rp1k_launch<8, 2, 2, 2>(a, s);
    case 5: return rp1k_launch<8, 2, 4, 2>(a, s);
    case 6: return rp1k_launch<16, 1, 2, 4>(a, s);
    case 7: return rp1k_launch<16, 2, 2, 4>(a, s);
    case 8: return rp1k_launch<32, 1, 1, 8>(a, s);
    case 9: return rp1k_launch<32, 2, 1, 8>(a, s);
    default: return HAWQ_ERR_UNSUPPORTED;
    }
}

}  // namespace hawq
