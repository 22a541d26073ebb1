// Tiled implicit GEMM for the large launches whose channel counts or operands the other tiled kernel (conv_mfma.hip) does not
// suit: input channels a multiple of 16 only (packed 4-bit: of 32), any number of output channels, unsigned bytes above 127, INT32
// results; and the middling ones, a few 64 x 64 tiles per CU.  The matrix product of hawq_gemm_int, the convolutions of
// Inception-style modules, residual networks' layers at small and middling batches.
//
// Two things differ from conv_mfma.hip.  Pixels are the MFMA's row operand and channels its column operand, so a lane holds one
// output channel and sixteen pixels: its parameters are a handful of registers, and a store instruction writes 32 consecutive
// channels of two pixels whatever the row's alignment (the other way round a lane's run of 16 channels needs whole, aligned groups).
// And a K-step is 64 bytes of the flattened (r, s, c) reduction index, of which a lane of an LDS-DMA fetch takes one 16-byte chunk and
// finds its filter tap with two multiplications (TAPS; one division per step and lane, whatever the number of rows it fetches).
//
// Operands travel global -> LDS by DMA into a ring of four stages, three steps ahead; a row's four chunks are XOR-swizzled with
// (row >> 2) & 3 on the source side, which makes every fragment read free of bank conflicts.  One barrier per step.  Chunks past
// the reduction's end read as zeros on the pixel side, so what the weight side then holds does not matter.
//
// RES, DUAL: an identity shortcut, read as the results are stored; a second convolution (1x1) whose steps follow the first one's, with
// sums of its own.  XF: unsigned bytes above 127 are multiplied as x - 128 (one XOR per dword of a fragment); 128 times the sum of a channel's weights
// is added at the end, the sums formed by dot products on the vector ALU from the fragments the MFMAs read (so that padding and
// ragged ends cancel exactly).  FORM 1: packed 4-bit operands, split into nibbles between fragment read and MFMA, weights kept as 16 w.
//
// Bound: matrix cores and the 64 B/clk a CU's vector-memory path delivers, in balance for a 128 x 128 tile.  Against the
// split-reduction kernel that took these launches: 4096 x 4096 x 4096 unsigned bytes to INT32 263 -> 78 us (1.76 POP/s), to bytes 274
// -> 75, 4096 x 1000 x 1024 28 -> 11; 35 x 35 at batch 32: 1x1 288 -> 64 packed 4-bit 13.7 -> 6.1, 3x3 96 -> 96 8-bit 19.4 -> 12.3, 1x1
// 288 -> 288 42.5 -> 16.5.  Against conv_mfma.hip, signed bytes: 1024 x 1000 x 256 to INT32 15.5 -> 3.9 (its element-wise epilogue),
// 4096 x 4096 x 4096 to bytes 96 -> 68.
#include "common.h"
#include "fastdiv.h"

namespace hawq {

struct TileArgs {
    FastDiv ch, S, PQ, Q;   // 16-byte chunks of a tap, filter width, output pixels of an image, output width
    uint32_t n_nt;          // channel tiles
    int32_t vec;            // whole groups of four channels and an aligned output: dword stores of 8-bit results
};

// BM x BN (pixels x channels) per workgroup of WM x WN waves
template <int BM, int BN, int WM, int WN, int FORM, bool XF, bool TAPS, bool RES, bool DUAL>
__global__ void __launch_bounds__(WM *WN * 64) __attribute__((amdgpu_waves_per_eu(BM * BN / (WM * WN) >= 64 * 64 ? 2 : 3)))
conv_tile_kernel(const ConvArgs a, const TileArgs e) {
    constexpr int NW = WM * WN;                             // waves
    constexpr int TM = BM / WM / 32, TN = BN / WN / 32;     // 32 x 32 tiles of a wave
    constexpr int IX = BM / 16, IW = BN / 16;               // fetch instructions (16 rows, 1 KB) of a stage
    constexpr int NX = IX / NW, NB = IW / NW;               // ... of a wave
    constexpr int NL = NX + NB;
    static_assert(IX % NW == 0 && IW % NW == 0 && NX > 0 && NB > 0, "every wave fetches equally");
    constexpr int NBUF = 4, STAGE = (BM + BN) * 64;
    constexpr uint32_t kInvalid = 0x80000000u;
    __shared__ __attribute__((aligned(1024))) uint8_t lds0[STAGE];
    __shared__ __attribute__((aligned(1024))) uint8_t lds1[STAGE];
    __shared__ __attribute__((aligned(1024))) uint8_t lds2[STAGE];
    __shared__ __attribute__((aligned(1024))) uint8_t lds3[STAGE];
    auto buf = [&](auto nc) -> uint8_t * {   // (separate objects: the compiler tracks asynchronous LDS writes per object)
        constexpr int n = decltype(nc)::value % NBUF;
        if constexpr (n == 0) return lds0;
        else if constexpr (n == 1) return lds1;
        else if constexpr (n == 2) return lds2;
        else return lds3;
    };
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const uint32_t L = xcd_remap(blockIdx.x, gridDim.x);
    const int m0 = (int)(L / e.n_nt) * BM, n0 = (int)(L % e.n_nt) * BN;

    const int Cb = FORM == 0 ? a.C : a.C / 2;
    const int n_ch = Cb >> 4, n_chunks = a.R * a.S * n_ch, steps = (n_chunks + 3) >> 2;
    const int row_b = n_chunks * 16;
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, a.N * a.H * a.W * Cb, 0x00020000);
    // weights: [K][row], or -- every K-step a whole 64-byte block -- the blocked copy, contiguous per step (see ConvArgs::w_t)
    const bool tiled = a.w_t != nullptr;
    const int wstep = tiled ? 4096 : 64;
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)(tiled ? a.w_t : a.w), 0, tiled ? (a.K + 63) / 64 * steps * 4096 : a.K * row_b, 0x00020000);

    // DUAL: the steps after the main branch's are the shortcut convolution's, a 1x1 window without padding
    const int Csb = DUAL ? (FORM == 0 ? a.Cs : a.Cs / 2) : 0;
    const int n_chs = Csb >> 4, steps_s = (n_chs + 3) >> 2, total = steps + steps_s;
    const __amdgpu_buffer_rsrc_t rs_xs = __builtin_amdgcn_make_buffer_rsrc((void *)(DUAL ? a.xs : a.x), 0, DUAL ? a.N * a.Hs * a.Ws * Csb : 0, 0x00020000);
    const bool tiled_s = DUAL && a.ws_t != nullptr;
    const __amdgpu_buffer_rsrc_t rs_ws = __builtin_amdgcn_make_buffer_rsrc((void *)(DUAL ? (tiled_s ? a.ws_t : a.ws) : a.w), 0, tiled_s ? (a.K + 63) / 64 * steps_s * 4096 : a.K * Csb, 0x00020000);

    // ---- this lane's rows of a stage: instruction i fills rows 16 i .. 16 i + 15, four lanes each ----
    const int c4 = (lane & 3) ^ ((lane >> 4) & 3);          // the chunk the swizzle places at the lane's position
    uint32_t xoff[NX], woff[NB], xsoff[DUAL ? NX : 1], wsoff[DUAL ? NB : 1];
    int ih0[NX], iw0[NX];
#pragma unroll
    for (int j = 0; j < NX; ++j) {
        const uint32_t m = (uint32_t)(m0 + (j * NW + wave) * 16 + (lane >> 2));
        const uint32_t nn = fdiv(m, e.PQ), pq = m - nn * (uint32_t)(a.P * a.Q);
        const uint32_t p = fdiv(pq, e.Q), q = pq - p * (uint32_t)a.Q;
        ih0[j] = (int)p * a.stride_h - a.pad_h;
        iw0[j] = (int)q * a.stride_w - a.pad_w;
        xoff[j] = (uint32_t)((((int)nn * a.H + ih0[j]) * a.W + iw0[j]) * Cb);
        if (m >= (uint32_t)a.M) {
            if (TAPS) ih0[j] = 1 << 30;                     // (fails the bounds test of every tap)
            else xoff[j] = kInvalid;
        }
        if constexpr (DUAL)
            xsoff[j] = m >= (uint32_t)a.M ? kInvalid : (uint32_t)((((int)nn * a.Hs + (int)p * a.stride_sh) * a.Ws + (int)q * a.stride_sw) * Csb);
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int n = n0 + (j * NW + wave) * 16 + (lane >> 2);
        woff[j] = n >= a.K ? kInvalid : tiled ? (uint32_t)((n >> 6) * steps * 4096 + (n & 63) * 64 + c4 * 16) : (uint32_t)(n * row_b + c4 * 16);
        if constexpr (DUAL)
            wsoff[j] = n >= a.K ? kInvalid : tiled_s ? (uint32_t)((n >> 6) * steps_s * 4096 + (n & 63) * 64 + c4 * 16) : (uint32_t)(n * Csb + c4 * 16);
    }
    auto fetch = [&](int step, auto bc) {
        if (DUAL && step >= steps) {
            if constexpr (DUAL) {
                const uint32_t ks = (uint32_t)((step - steps) * 4 + c4);
#pragma unroll
                for (int j = 0; j < NX; ++j)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_xs, (__attribute__((address_space(3))) void *)(buf(bc) + (j * NW + wave) * 1024), 16,
                                                             (int)(ks < (uint32_t)n_chs && xsoff[j] != kInvalid ? xsoff[j] + ks * 16 : kInvalid), 0, 0, 0);
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_ws, (__attribute__((address_space(3))) void *)(buf(bc) + BM * 64 + (j * NW + wave) * 1024), 16,
                                                             (int)(wsoff[j] == kInvalid ? kInvalid : wsoff[j] + (step - steps) * (tiled_s ? 4096 : 64)), 0, 0, 0);
            }
            return;
        }
        const uint32_t kc = (uint32_t)(step * 4 + c4);
        const bool in = kc < (uint32_t)n_chunks;
        uint32_t off, r = 0, s = 0;
        if constexpr (TAPS) {
            const uint32_t tap = fdiv(kc, e.ch);
            r = fdiv(tap, e.S);
            s = tap - r * (uint32_t)a.S;
            off = (r * (uint32_t)a.W + s) * (uint32_t)Cb + (kc - tap * (uint32_t)n_ch) * 16;
        } else {
            off = kc * 16;
        }
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            const bool ok = TAPS ? in & ((uint32_t)(ih0[j] + (int)r) < (uint32_t)a.H) & ((uint32_t)(iw0[j] + (int)s) < (uint32_t)a.W)
                                 : in & (xoff[j] != kInvalid);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (__attribute__((address_space(3))) void *)(buf(bc) + (j * NW + wave) * 1024), 16,
                                                     (int)(ok ? xoff[j] + off : kInvalid), 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j)   // (past the reduction's end: the next rows or, past the last, zeros)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, (__attribute__((address_space(3))) void *)(buf(bc) + BM * 64 + (j * NW + wave) * 1024), 16,
                                                     (int)(woff[j] == kInvalid ? kInvalid : woff[j] + step * wstep), 0, 0, 0);
    };
    static_for<0, NBUF - 1>([&](auto ic) { fetch(decltype(ic)::value, ic); });

    // ---- the shortcut, in the form the results are stored in: of pixel 8 j + 4 half + q, the four channels of the lane's quad ----
    const int col = lane & 31, half = lane >> 5;
    const int q = lane & 3;                               // position in its quad of lanes = of four consecutive channels
    uint32_t resw[RES ? TM : 1][RES ? TN : 1][4];
    if constexpr (RES) {
        const bool r4 = is4(a.res_dt);
        const __amdgpu_buffer_rsrc_t rs_r = __builtin_amdgcn_make_buffer_rsrc((void *)a.res, 0, (int)tensor_bytes((int64_t)a.M * a.K, a.res_dt), 0x00020000);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm)
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) {
                const int ch4 = n0 + (wn * TN + tn) * 32 + (col & ~3);
                const uint32_t o = (uint32_t)(m0 + (wm * TM + tm) * 32 + 4 * half + q) * (uint32_t)a.K + (uint32_t)ch4;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t at = ch4 < a.K ? o + (uint32_t)(8 * j * a.K) : kInvalid;
                    if (r4) {
                        const uint32_t h = __builtin_amdgcn_raw_buffer_load_b16(rs_r, (int)(ch4 < a.K ? at >> 1 : kInvalid), 0, 0);
                        resw[tm][tn][j] = (h & 0xfu) | ((h & 0xf0u) << 4) | ((h & 0xf00u) << 8) | ((h & 0xf000u) << 12);
                    } else {
                        resw[tm][tn][j] = __builtin_amdgcn_raw_buffer_load_b32(rs_r, (int)at, 0, 0);
                    }
                }
            }
    }
    // ---- the lane's channels' parameters ----
    int32_t bias[TN], pb[TN], pcs[TN], prb[TN], prc[TN], sbias[DUAL ? TN : 1], sb[DUAL ? TN : 1], scs[DUAL ? TN : 1];
    const bool mid = DUAL && a.mid_s8;                    // the shortcut's own INT8 result, rescaled once more
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        const int ch = n0 + (wn * TN + tn) * 32 + col;
        bias[tn] = ch < a.K ? a.bias[ch] : 0;
        pb[tn] = a.b != nullptr && ch < a.K ? a.b[ch] : 0;
        pcs[tn] = a.b != nullptr && ch < a.K ? a.c[ch] : 1;
        if constexpr (RES) {
            prb[tn] = ch < a.K ? a.res_b[ch] : 0;
            prc[tn] = ch < a.K ? a.res_c[ch] : 1;
        }
        if constexpr (DUAL) {
            sbias[tn] = ch < a.K ? a.bias_s[ch] : 0;
            sb[tn] = ch < a.K ? a.b_s[ch] : 0;
            scs[tn] = ch < a.K ? a.c_s[ch] : 1;
            prb[tn] = mid && ch < a.K ? a.res_b[ch] : 0;
            prc[tn] = mid && ch < a.K ? a.res_c[ch] : 1;
        }
    }

    // ---- fragment addresses within a stage ----
    int xf[TM][2], wf[TN][2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) {
            const int row = (wm * TM + tm) * 32 + col;
            xf[tm][kk] = row * 64 + (((kk * 2 + half) ^ ((row >> 2) & 3)) << 4);
        }
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            const int row = (wn * TN + tn) * 32 + col;
            wf[tn][kk] = BM * 64 + row * 64 + (((kk * 2 + half) ^ ((row >> 2) & 3)) << 4);
        }
    }
    v16i acc[TM][TN], accm[DUAL ? TM : 1][DUAL ? TN : 1];   // (DUAL: the main branch's sums move to accm when its steps are done)
    int32_t wsum[XF ? TN : 1] = {};
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[tm][tn][i] = 0;
    auto mul = [&](v4i(&x)[TM], const v4i(&w)[TN]) {
        if constexpr (XF) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) x[tm] ^= (int)0x80808080;
#pragma unroll
            for (int tn = 0; tn < TN; ++tn)
#pragma unroll
                for (int d = 0; d < 4; ++d) wsum[tn] = __builtin_amdgcn_sdot4(w[tn][d], 0x01010101, wsum[tn], false);
        }
        if constexpr (FORM == 0) {
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) acc[tm][tn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(x[tm], w[tn], acc[tm][tn], 0, 0, 0);
        } else {
            v4i wl[TN], wh[TN];
#pragma unroll
            for (int tn = 0; tn < TN; ++tn) { wl[tn] = (w[tn] << 4) & (int)0xF0F0F0F0; wh[tn] = w[tn] & (int)0xF0F0F0F0; }
#pragma unroll
            for (int tm = 0; tm < TM; ++tm) {
                const v4i xl = x[tm] & 0x0F0F0F0F, xh = (x[tm] >> 4) & 0x0F0F0F0F;
#pragma unroll
                for (int tn = 0; tn < TN; ++tn) {
                    acc[tm][tn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xl, wl[tn], acc[tm][tn], 0, 0, 0);
                    acc[tm][tn] = __builtin_amdgcn_mfma_i32_32x32x32_i8(xh, wh[tn], acc[tm][tn], 0, 0, 0);
                }
            }
        }
    };
    // Step t: its second-half fragments are read, step t + 3 is requested into the stage that step t - 1 has left, the first half is
    // multiplied (its fragments were read during step t - 1), then the second half, with step t + 1's first-half fragments read
    // meanwhile.  At the closing barrier this wave's requests for step t + 2 have landed (only step t + 3's may fly) and its own
    // fragment reads are done.  The parameter loads above are older than any request waited for here.
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(0) : "memory");
    v4i x0[TM], w0[TN];
#pragma unroll
    for (int tm = 0; tm < TM; ++tm) x0[tm] = *(const v4i *)(lds0 + xf[tm][0]);
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) w0[tn] = *(const v4i *)(lds0 + wf[tn][0]);
    auto iteration = [&](int step, auto ic) {
        constexpr int ph = decltype(ic)::value;
        v4i x1[TM], w1[TN];
        if constexpr (DUAL) {
            if (step == steps) {
#pragma unroll
                for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                    for (int tn = 0; tn < TN; ++tn) {
                        accm[tm][tn] = acc[tm][tn];
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[tm][tn][i] = 0;
                    }
            }
        }
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) x1[tm] = *(const v4i *)(buf(ic) + xf[tm][1]);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) w1[tn] = *(const v4i *)(buf(ic) + wf[tn][1]);
        fetch(step + NBUF - 1, std::integral_constant<int, ph + NBUF - 1>{});
        mul(x0, w0);
#pragma unroll
        for (int tm = 0; tm < TM; ++tm) x0[tm] = *(const v4i *)(buf(std::integral_constant<int, ph + 1>{}) + xf[tm][0]);
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) w0[tn] = *(const v4i *)(buf(std::integral_constant<int, ph + 1>{}) + wf[tn][0]);
        mul(x1, w1);
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(NL) : "memory");
    };
    for (int step = 0;; step += NBUF) {
        iteration(step, std::integral_constant<int, 0>{});
        if (step + 1 >= total) break;
        iteration(step + 1, std::integral_constant<int, 1>{});
        if (step + 2 >= total) break;
        iteration(step + 2, std::integral_constant<int, 2>{});
        if (step + 3 >= total) break;
        iteration(step + 3, std::integral_constant<int, 3>{});
        if (step + 4 >= total) break;
    }

    // ---- epilogue: a lane has channel `col` of each tile and, of half h, pixels 8 j + 4 h + k (register 4 j + k) ----
    const bool rq = a.b != nullptr;
    bool narrow = true;
    int32_t bs[TN], ss[DUAL ? TN : 1];
#pragma unroll
    for (int tn = 0; tn < TN; ++tn) {
        if constexpr (XF) {
            wsum[tn] += __shfl_xor(wsum[tn], 32);
            bias[tn] += 128 * wsum[tn];
        }
        narrow &= pcs[tn] <= 32 && ((uint32_t)pb[tn] >> ((pcs[tn] - 1) & 31)) == 0;
        bs[tn] = (int32_t)((uint32_t)pb[tn] << ((32 - pcs[tn]) & 31));
        if constexpr (RES) narrow &= prc[tn] <= 31 && (uint32_t)prb[tn] < 1u << 22;   // (r rb + 2^(rc-1)) >> rc in 32 bits
        if constexpr (DUAL) {
            narrow &= scs[tn] <= 32 && ((uint32_t)sb[tn] >> ((scs[tn] - 1) & 31)) == 0 && prc[tn] <= 31 && (uint32_t)prb[tn] < 1u << 22;
            ss[tn] = (int32_t)((uint32_t)sb[tn] << ((32 - scs[tn]) & 31));
        }
    }
    narrow = __all(narrow);
    int32_t lo = a.lo, hi = a.hi;
    int64_t round = (int64_t)1 << 31;
    asm volatile("" : "+v"(lo), "+v"(hi), "+v"(round));   // (opaque addend and bounds: one multiply-add, one median per output)
    const int y_dt = a.y_dt, K = a.K;
    const __amdgpu_buffer_rsrc_t rs_y = __builtin_amdgcn_make_buffer_rsrc((void *)a.y, 0, (int)tensor_bytes((int64_t)a.M * K, y_dt), 0x00020000);
    // four x four bytes change places within a quad of lanes: byte k of lane q <-> byte q of lane k
    const uint32_t sel01 = (uint32_t)(q | (4 + q) << 8) | 0x0c0c0000u, sel23 = (uint32_t)(q << 16 | (4 + q) << 24) | 0x00000c0cu;
    auto quad_transpose = [&](uint32_t p) -> uint32_t {
        const uint32_t t0 = (uint32_t)__builtin_amdgcn_mov_dpp((int)p, 0x00, 0xf, 0xf, true);
        const uint32_t t1 = (uint32_t)__builtin_amdgcn_mov_dpp((int)p, 0x55, 0xf, 0xf, true);
        const uint32_t t2 = (uint32_t)__builtin_amdgcn_mov_dpp((int)p, 0xaa, 0xf, 0xf, true);
        const uint32_t t3 = (uint32_t)__builtin_amdgcn_mov_dpp((int)p, 0xff, 0xf, 0xf, true);
        return __builtin_amdgcn_perm(t1, t0, sel01) | __builtin_amdgcn_perm(t3, t2, sel23);
    };
    const bool res_signed = RES && a.res_dt == HAWQ_S8;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            v16i v = DUAL ? accm[DUAL ? tm : 0][DUAL ? tn : 0] : acc[tm][tn];
            v16i u = acc[tm][tn];                         // (DUAL: the shortcut's sums)
            uint32_t rw[4] = {0, 0, 0, 0};                // shortcut bytes of the lane's channel, pixels 8 j + 4 half + 0 .. 3
            if constexpr (RES)
#pragma unroll
                for (int j = 0; j < 4; ++j) rw[j] = quad_transpose(resw[tm][tn][j]);
            if constexpr (FORM != 0) v >>= 4;
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] += bias[tn];
            if constexpr (DUAL) {
                if constexpr (FORM != 0) u >>= 4;
#pragma unroll
                for (int i = 0; i < 16; ++i) u[i] += sbias[tn];
            }
            if (rq) {
                if (__builtin_expect(narrow, 1)) {
                    int32_t s = bs[tn];
                    asm volatile("" : "+v"(s));           // (a hoisted 64-bit sign extension would make it a 64 x 32 product)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        int32_t y = (int32_t)(((int64_t)v[i] * (int64_t)s + round) >> 32);
                        if constexpr (RES) {
                            const int32_t r = res_signed ? __builtin_amdgcn_sbfe((int32_t)rw[i >> 2], 8 * (i & 3), 8) : (int32_t)__builtin_amdgcn_ubfe(rw[i >> 2], 8 * (i & 3), 8);
                            y += (__mul24(r, prb[tn]) + (int32_t)(1u << ((prc[tn] - 1) & 31))) >> prc[tn];
                        }
                        if constexpr (DUAL) {
                            int32_t z = ss[tn];
                            asm volatile("" : "+v"(z));
                            int32_t r = (int32_t)(((int64_t)u[i] * (int64_t)z + round) >> 32);
                            if (mid) {
                                r = r < -128 ? -128 : r > 127 ? 127 : r;
                                r = (__mul24(r, prb[tn]) + (int32_t)(1u << ((prc[tn] - 1) & 31))) >> prc[tn];
                            }
                            y += r;
                        }
                        asm("v_med3_i32 %0, %1, %2, %3" : "=v"(v[i]) : "v"(y), "v"(lo), "v"(hi));
                    }
                } else {
#pragma unroll 1
                    for (int i = 0; i < 16; ++i) {        // element 0, then all move down by one
                        int64_t w = rq64(v[0], pb[tn], pcs[tn]);
                        if constexpr (RES) {
                            w += rq64(res_signed ? (int32_t)(int8_t)rw[0] : (int32_t)(rw[0] & 0xff), prb[tn], prc[tn]);
                            rw[0] = rw[0] >> 8 | rw[1] << 24; rw[1] = rw[1] >> 8 | rw[2] << 24;
                            rw[2] = rw[2] >> 8 | rw[3] << 24; rw[3] >>= 8;
                        }
                        if constexpr (DUAL) {
                            int64_t r = rq64(u[0], sb[tn], scs[tn]);
                            if (mid) r = rq64(clamp64(r, -128, 127), prb[tn], prc[tn]);
                            w += r;
                            u = __builtin_shufflevector(u, u, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 0);
                        }
                        const int32_t y = clamp64(w, a.lo, a.hi);
                        v = __builtin_shufflevector(v, v, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 0);
                        v[15] = y;
                    }
                }
            }
            const int mb = m0 + (wm * TM + tm) * 32 + 4 * half;    // the lane's pixel of register 0
            const int ch = n0 + (wn * TN + tn) * 32 + col;
            // (rows past the last pixel lie past the buffer's end and are dropped; so are the channels marked here)
            if (y_dt == HAWQ_S32) {
                const uint32_t o = ch < K ? ((uint32_t)mb * (uint32_t)K + (uint32_t)ch) * 4 : kInvalid;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)v[i], rs_y, (int)(o + (uint32_t)((8 * (i >> 2) + (i & 3)) * K) * 4), 0, 0);
            } else if (!is4(y_dt) && !e.vec) {
                const uint32_t o = ch < K ? (uint32_t)mb * (uint32_t)K + (uint32_t)ch : kInvalid;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)v[i], rs_y, (int)(o + (uint32_t)((8 * (i >> 2) + (i & 3)) * K)), 0, 0);
            } else {
                // a lane then has the four channels of its quad, of pixel q
                const int ch4 = ch & ~3;
                const uint32_t o = (uint32_t)(mb + q) * (uint32_t)K + (uint32_t)ch4;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t p = __builtin_amdgcn_perm((uint32_t)v[4 * j + 1], (uint32_t)v[4 * j], 0x0c0c0400u) |
                                       __builtin_amdgcn_perm((uint32_t)v[4 * j + 3], (uint32_t)v[4 * j + 2], 0x04000c0cu);
                    const uint32_t w = quad_transpose(p);
                    const uint32_t at = o + (uint32_t)(8 * j * K);
                    if (!is4(y_dt)) {
                        __builtin_amdgcn_raw_buffer_store_b32(w, rs_y, (int)(ch4 < K ? at : kInvalid), 0, 0);
                    } else {
                        const uint32_t h = (w & 0xfu) | ((w >> 4) & 0xf0u) | ((w >> 8) & 0xf00u) | ((w >> 12) & 0xf000u);
                        if (e.vec) {
                            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)h, rs_y, (int)(ch4 < K ? at >> 1 : kInvalid), 0, 0);
                        } else {                          // (K is even)
                            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)h, rs_y, (int)(ch4 < K ? at >> 1 : kInvalid), 0, 0);
                            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(h >> 8), rs_y, (int)(ch4 + 2 < K ? (at >> 1) + 1 : kInvalid), 0, 0);
                        }
                    }
                }
            }
        }
}

// ---- host side ----

bool conv_tile_eligible(const ConvArgs &a, int x_hi) {
    const bool four = is4(a.x_dt);
    if (a.C % (four ? 32 : 16) != 0 || four != is4(a.w_dt) || a.xs != nullptr) return false;
    if (four ? (a.x_dt != HAWQ_U4 || a.w_dt != HAWQ_S4) : (a.w_dt != HAWQ_S8 || (a.x_dt != HAWQ_U8 && a.x_dt != HAWQ_S8))) return false;
    if (((uintptr_t)a.x | (uintptr_t)a.w) & 15) return false;
    if (((uintptr_t)a.bias | (uintptr_t)a.b) & 3) return false;
    if (a.y_dt == HAWQ_S32 && ((uintptr_t)a.y & 3)) return false;
    // a shortcut: whole groups of four channels on both sides, operands within the signed range
    if (a.res != nullptr && (a.b == nullptr || a.K % 4 != 0 || (((uintptr_t)a.res | (uintptr_t)a.y) & 3) || ((uintptr_t)a.res_b & 3) ||
                             a.res_dt == HAWQ_S4 || a.y_dt == HAWQ_S32 || (a.x_dt == HAWQ_U8 && x_hi > 127))) return false;
    const int64_t red = (int64_t)a.R * a.S * a.C;
    // packed sums are kept times sixteen (16 * 15 * 8 * red < 2^31), chunk numbers (red / 16 and some steps) well below 2^31, rows of
    // the tiles that reach past M * K and offsets past a row's last chunk below the mark of an invalid one
    if (red >= (four ? 1 << 20 : 1 << 22) || (int64_t)a.H + a.R >= (1 << 29) || (int64_t)a.W + a.S >= (1 << 29)) return false;
    const int64_t edge = (int64_t)1 << 31;
    if (((int64_t)a.M + 256) * a.K * (a.y_dt == HAWQ_S32 ? 4 : 1) >= edge || (int64_t)(a.K + 64) * (red + 64) + 65536 >= edge) return false;
    return (int64_t)a.N * a.H * a.W * a.C + 4 * red < edge;
}

bool conv_tile_dual_eligible(const ConvArgs &a, int x_hi, int xs_hi) {
    if (a.xs == nullptr || a.res != nullptr || a.b == nullptr || a.y_dt == HAWQ_S32 || a.K % 4 != 0) return false;
    if (a.mid_s8 && (a.res_b == nullptr || a.res_c == nullptr)) return false;
    ConvArgs m = a, t = a;                                  // each branch as a layer of its own
    m.xs = t.xs = nullptr;
    t.x = a.xs; t.w = a.ws; t.bias = a.bias_s; t.b = a.b_s; t.H = a.Hs; t.W = a.Ws; t.C = a.Cs; t.R = t.S = 1; t.x_dt = a.xs_dt; t.w_dt = a.ws_dt;
    if (is4(a.x_dt) != is4(a.xs_dt) || (a.x_dt == HAWQ_U8 && x_hi > 127) || (a.xs_dt == HAWQ_U8 && xs_hi > 127)) return false;
    if (((uintptr_t)a.y | (uintptr_t)a.bias_s | (uintptr_t)a.b_s | (uintptr_t)(a.mid_s8 ? a.res_b : nullptr)) & 3) return false;
    return conv_tile_eligible(m, x_hi) && conv_tile_eligible(t, xs_hi);
}

template <int BM, int BN, int WM, int WN, bool RES, bool DUAL = false>
static hawq_status tile_launch(const ConvArgs &a, TileArgs e, int x_hi, hipStream_t s) {
    e.n_nt = (a.K + BN - 1) / BN;
    const uint32_t nb = e.n_nt * (uint32_t)((a.M + BM - 1) / BM);
    constexpr int T = WM * WN * 64;
    const bool xf = a.x_dt == HAWQ_U8 && x_hi > 127, taps = a.R * a.S > 1 || a.pad_h != 0 || a.pad_w != 0;
    auto go = [&](auto kernel) { kernel<<<nb, T, 0, s>>>(a, e); };
    if constexpr (DUAL) {
        if (is4(a.x_dt)) taps ? go(conv_tile_kernel<BM, BN, WM, WN, 1, false, true, false, true>) : go(conv_tile_kernel<BM, BN, WM, WN, 1, false, false, false, true>);
        else taps ? go(conv_tile_kernel<BM, BN, WM, WN, 0, false, true, false, true>) : go(conv_tile_kernel<BM, BN, WM, WN, 0, false, false, false, true>);
    } else if (is4(a.x_dt)) taps ? go(conv_tile_kernel<BM, BN, WM, WN, 1, false, true, RES, false>) : go(conv_tile_kernel<BM, BN, WM, WN, 1, false, false, RES, false>);
    else if constexpr (!RES) {
        if (xf) taps ? go(conv_tile_kernel<BM, BN, WM, WN, 0, true, true, RES, false>) : go(conv_tile_kernel<BM, BN, WM, WN, 0, true, false, RES, false>);
        else taps ? go(conv_tile_kernel<BM, BN, WM, WN, 0, false, true, RES, false>) : go(conv_tile_kernel<BM, BN, WM, WN, 0, false, false, RES, false>);
    } else taps ? go(conv_tile_kernel<BM, BN, WM, WN, 0, false, true, RES, false>) : go(conv_tile_kernel<BM, BN, WM, WN, 0, false, false, RES, false>);
    return check_launch();
}

// Tiles BM x BN and an estimate of a launch's time with them, in units of 0.01 us beyond what all share.  A step takes at least what
// a workgroup alone on its CU needs for it (its chain of landing wait, barrier, fragment reads and MFMAs), and per CU the time
// to draw its tiles' operands from behind the L2s, 50 KB/us; the epilogue comes on top.  Fitted to 4096 x 4096 x 4096 down to
// 300 x 100 x 256 and module convolutions, where the choice is within 5 % of the best of the five almost everywhere: 4096 x 4096 x 4096
// 256 x 256 tiles 68 us (128 x 128 97, 64 x 64 171), 4096 x 1000 x 4096 128 x 128 24 (256 x 256 44, 64 x 64 41), 1024 x 1000 x 4096 64 x 64
// 16.6 (128 x 128 21, 64 x 32 16.9), 300 x 1003 x 1024 64 x 32 4.5 (64 x 64 4.5, 128 x 64 5.7).
struct TileCfg { int32_t bm, bn, chain; };
constexpr TileCfg kTile[] = {{256, 256, 75}, {128, 128, 37}, {128, 64, 27}, {64, 64, 20}, {64, 32, 17}};

static int64_t tile_steps(const ConvArgs &a) { return ((int64_t)a.R * a.S * (is4(a.x_dt) ? a.C / 2 : a.C) + 63) / 64; }
static int tile_choice(const ConvArgs &a) {
    const int64_t steps = tile_steps(a);
    int best = 0;
    int64_t cost = INT64_MAX;
    for (int i = 0; i < 5; ++i) {
        const TileCfg &t = kTile[i];
        const int64_t per_cu = (((int64_t)a.M + t.bm - 1) / t.bm * ((a.K + t.bn - 1) / t.bn) + 255) / 256;
        const int64_t draw = per_cu * (t.bm + t.bn) * 64 / 512;   // 0.01 us a step
        const int64_t c = steps * (draw > t.chain ? draw : t.chain) + per_cu * t.bm * t.bn / 150;
        if (c < cost) { cost = c; best = i; }
    }
    return best;
}

static int64_t tiles_of(const ConvArgs &a, int bm, int bn) { return ((int64_t)a.M + bm - 1) / bm * ((a.K + bn - 1) / bn); }

// A handful of output channels, a long 3x3 or 1x1 reduction and very many pixels: most of a 32-channel tile's products are for nothing,
// and this kernel fetches more for them than the other two (3x3 592 -> 8 at 90944 pixels 70 us, the split-reduction kernel 54; 512 -> 10
// at 122304 74 and, conv_mfma.hip, 53; with fewer pixels it is no slower: 560 -> 11 at 68502 42.8 and 48.5).  From 58 steps on with still more
// pixels (448 -> 10 at 107800 57.7 and, conv_mfma.hip, 46; 432 -> 12 at 98049 45 and 38.7; over 117 layers of 59 to 63 steps
// above that line the others need 0.94 of this kernel's time).
static bool tile_narrow(const ConvArgs &a) {
    return !is4(a.x_dt) && a.K <= 12 && a.R * a.S <= 9 && tiles_of(a, 64, 64) >= (tile_steps(a) >= 64 ? 1280 : tile_steps(a) >= 58 ? 1500 : INT64_MAX);
}

// Over the split-reduction kernel below its line of 2^19 outputs: matrix products and 1x1 layers of no more than 24 steps.  From
// 2^18 outputs on with 8-bit operands and 8 steps or more, or with ragged rows (300 x 1000 x 1024 6.7 -> 4.6 us, 300 x 1003 x 256 4.9 ->
// 3.4; with 64 steps 14.4 and 15.1), from 3 * 2^17 on with fewer (8670 pixels of packed 288 -> 48 4.6 -> 4.2; 7350 3.8 and 4.1).  Packed
// operands stay there while its 32 x 64 tiles are no more than one to a CU (3136 pixels of 448 -> 132 3.8 us, here 4.4; 2450 of
// 704 -> 176 4.3 and 4.9; above that 0.92 of its time in the mean of 85 shapes), but for ragged rows of one or two steps (4900 of
// 128 -> 66 4.0 and 3.7).  A 3x3 window stays there (4624 pixels of 64 -> 96 4.2 us, here 5.8), and so do longer packed reductions (1024 ->
// 2048 / 2 at 196 pixels 5.3 us, here 6.3; 2048 -> 512 at 784 7.4 and 8.2).  8-bit reductions of more than 64 steps over a few channels
// come here with more than two rounds of tiles (5x5 / 2 416 -> 7 at 34496 pixels 84 -> 54 us; 3x3 496 -> 4 at 35258 28.3 -> 21.8), with many
// more of them they stay (5x5 608 -> 3 at 98980 132 us, here 174).
bool conv_tile_over_sk(const ConvArgs &a) {
    if (a.res != nullptr) return false;
    const bool four = is4(a.x_dt);
    const int64_t out = (int64_t)a.M * a.K, steps = tile_steps(a);
    if (!four && steps > 64 && tiles_of(a, 64, 64) > 512) return tiles_of(a, 64, 64) <= 896;
    const bool ragged = a.K % 4 != 0;
    const bool round = four && tiles_of(a, 64, 32) <= 256 && (steps >= 3 || !ragged);
    if (a.R * a.S != 1 || steps > 24 || round || (four && steps >= 8 && !ragged)) return false;
    return out > (steps >= 8 || ragged ? 1 << 18 : 3 << 17);
}

// Launches of no more than two or three 64 x 64 tiles per CU: those tiles, three workgroups side by side on a CU, whose fetches,
// products and epilogues overlap (shortcut, 64 -> 256 at 56 x 56, packed, batch 2: 5.0 us, with 128 x 64 6.2; 3x3 / 2 64 -> 128, batch
// 16: 6.2 and 6.6).  With more tiles or steps the larger tiles' fewer bytes count (512 x 4096 x 4096 22.7 us, with 64 x 64 23.8; shortcut,
// packed 3x3 256 -> 256 at 14 x 14, batch 48, 588 tiles of 18 steps: 16.9, conv_mfma.hip 16.4).
// Beside another part's kernels (corun) the same: with and without the larger tiles there ResNet50 at batch 96, 128, 192 and 256 takes 875
// and 880 us, 1038 and 1038, 1475 and 1468, 1812 and 1808, mixed at 256 1783 and 1776, ResNet18 at 128 367 and 369, all within what
// two runs of one side differ by.
static bool few_tiles(const ConvArgs &a) {
    const int64_t steps = tile_steps(a), tiles = tiles_of(a, 64, 64);
    return tiles <= (steps < 16 ? 768 : steps < 32 ? 512 : 0);
}

// Over the tiled kernel with pixels along the lanes (mfma: that kernel takes the launch) or, above its line, the split-reduction
// kernel.  The former's tiles are 128 channels wide and its workgroups of eight waves, one or two on a CU: a launch of few tiles is
// faster here (56 x 56, 64 -> 256 with its shortcut, batch 1, 5.7 -> 3.9 us, batch 4 5.6 and 5.6; packed 3x3 / 2 64 -> 128, batch 8 9.1 ->
// 5.3; packed 3x3 256 -> 256 at 14 x 14 with its shortcut, batch 16 14.2 -> 9.7), from seven tiles of rows on (1024 -> 2048 / 2 at 196
// pixels 7.0 us, here 7.4; at 588 8.9 and 8.2) and for packed shortcut layers up to 1024 channels (512 -> 2048 at 784 pixels 7.5
// and 8.1; 256 -> 1024 at 784 5.9 and 5.3).  Of the larger launches it keeps those with whole groups of 16 channels, 8-bit
// results and no quarter of a 128-channel tile to spare, and every shortcut: its epilogue stores 16 bytes a lane (1x1 512 -> 128 at
// 28x28, batch 64 11.2 us, here 10.8; 3x3 / 2 256 -> 512 at 14x14, batch 128 13.3 and 14.8); this one takes INT32 results
// (4096 x 1000 x 256 25 -> 7.3), ragged ones (19 -> 5.5), 96 or 192 channels (3x3 64 -> 96 at 35x35, batch 32 12.9 -> 9.3) and products
// large enough for 256 x 256 tiles.  Of the launches of few tiles it keeps, too, shortcut layers of fewer than 1024 pixels, no more than
// a tile to a CU and more than 16 steps, packed 8 (3x3 384 -> 688 at 784 pixels, packed, 11.2 us, here 12.5; 192 -> 960 8.8 and 9.4), and 8-bit
// ones of more than two tiles a CU and 12 steps on whose weights have no blocked copy (1x1 896 -> 928 at 3136 pixels 7.5 and 8.9;
// 768 -> 704 6.7 and 7.5).
// The split-reduction kernel keeps long packed reductions just above its line (5x5 224 -> 112 at 7350 pixels 13.0 us, here 16.0; at
// 8670 24.3 and 20.2) and all of 13 steps or more, with a shortcut 8, whose 64 x 64 tiles are no more than one to a CU (3x3 224 -> 560 at
// 1225 pixels with a shortcut 8.0 us, here 9.3; 5x5 96 -> 576 8.0 and 8.7), and shortcuts of up to 16 channels, 8-bit 12 (packed
// 3x3 608 -> 8 at 159250 pixels 52 and 74, 8-bit 5x5 96 -> 4 at 194775 35 and 45, but 3x3 592 -> 16 at 43512 40 and 31).
bool conv_tile_preferred(const ConvArgs &a, bool mfma) {
    const bool four = is4(a.x_dt), res = a.res != nullptr;
    const int64_t steps = tile_steps(a), tiles = tiles_of(a, 64, 64), out = (int64_t)a.M * a.K;
    if (!res && tile_narrow(a)) return false;
    if (mfma) {
        const bool kept = (res && a.M < 1024 && tiles <= 256 && (four ? steps >= 8 && a.C % 128 == 0 : steps > 16)) ||
                          (!four && a.w_t == nullptr && a.K >= 128 && steps >= 12 && steps < 16 && tiles > 512);
        if (a.y_dt != HAWQ_S32 && a.M >= 448 && few_tiles(a) && !(four && res && a.K > 1024) && !(kept && a.K % 16 == 0)) return true;
        if (res) return false;
        if (a.K % 16 == 0 && a.M < 1024 && steps >= 32 && tiles <= 256) return false;
        return a.K % 16 != 0 || a.y_dt == HAWQ_S32 || (a.K > 64 && (a.K < 128 || (a.R * a.S == 1 && (a.K + 127) / 128 * 512 >= 5 * a.K))) || (steps >= 16 && tile_choice(a) == 0);
    }
    if (res && (four ? a.K <= 16 && steps >= 12 : a.K <= 12 && steps >= 25)) return false;
    if (four) return !((steps >= 20 && out <= 7 << 17) || (steps >= (res ? 8 : 13) && tiles <= 256));
    return !(steps >= 32 && out <= 5 << 17 && (steps <= 64 || tiles <= 512 || tiles > 896));
}

// Two convolutions in one launch.  Packed operands always, the direct kernel is what else takes them (56 x 56, 64 -> 256 plus 64, batch
// 1 267 us, here 5.4, batch 64 11700 and 63).  Bytes with few tiles, as few_tiles counts them over both branches' steps; conv_mfma.hip
// keeps a larger tile's sums twice and has one workgroup of it on a CU (56 x 56, 64 -> 256 plus 64, batch 1 8.2 -> 5.2 us; 28 x 28, 128 ->
// 512 plus 256 / 2, batch 2 9.5 -> 6.2, 8 10.6 -> 9.4; 3x3 256 -> 256 at 14 x 14 plus 128 / 2, batch 16 24.2 -> 19.1, 48 24.4 and 26.4),
// from 41 steps on up to 320 tiles (3x3 256 -> 512 plus 512 / 2 at 7 x 7, batch 53, 328 tiles of 44 steps 21.1 us, here 22.8).  Where
// the main branch's term fits 16 bits its eight-wave form is better than that: up to a tile per CU (ResNet50 at batch 1 223.4 ->
// 221.0 us, ResNet18 at 8 140.3 -> 138.1; at 32, with 392 tiles of 38 steps, 207 and 213).
// What conv_mfma.hip does not take (mfma: it does) comes here from more than one 64 x 64 tile to a CU on, below that with few steps: the
// split-reduction kernel is the other one, held up only by a long shortcut without blocked weights (up to 256 tiles of 17 to 20 steps
// 9.0 us here, 10.5 there; windows of 13 to 18 steps 9.0 to 10.2 and 7.3 to 7.7; of 25 to 64 steps 1.3 to 1.4 times its time; over
// 256 tiles 0.46 to 0.94 of it by steps and tiles, up to 1.1 with more than 32 steps; 700 shapes).
bool conv_tile_dual_preferred(const ConvArgs &a, bool mfma) {
    if (is4(a.x_dt)) return true;
    const int64_t steps = tile_steps(a) + (a.Cs + 63) / 64, tiles = tiles_of(a, 64, 64);
    if (!mfma) return tiles > 256 || steps <= (a.R * a.S > 1 || a.ws_t ? 12 : 20);
    return tiles <= (a.dual16 ? (steps < 32 ? 256 : 0) : steps < 16 ? 768 : steps < 41 ? 512 : steps < 64 ? 320 : 0);
}

hawq_status launch_conv_tile(const ConvArgs &a_in, int x_hi, hipStream_t s) {
    ConvArgs a = a_in;
    if (a.M == 0) return HAWQ_OK;
    if (a.C % (is4(a.x_dt) ? 128 : 64) != 0) a.w_t = nullptr;   // (the blocked copy holds whole 64-byte K-steps of one tap each)
    TileArgs e{};
    e.ch = fast_div((is4(a.x_dt) ? a.C / 2 : a.C) / 16);
    e.S = fast_div(a.S);
    e.PQ = fast_div(a.P * a.Q);
    e.Q = fast_div(a.Q);
    e.vec = a.K % 4 == 0 && ((uintptr_t)a.y & 3) == 0;
    if (a.xs != nullptr) {
        if (a.Cs % (is4(a.x_dt) ? 128 : 64) != 0) a.ws_t = nullptr;
        return tile_launch<64, 64, 2, 2, false, true>(a, e, x_hi, s);
    }
    if (a.res != nullptr) return tile_launch<64, 64, 2, 2, true>(a, e, x_hi, s);   // (one form: larger launches stay with conv_mfma.hip)
    const int choice = tile_choice(a);
    switch (choice < 3 && few_tiles(a) ? 3 : choice) {
    case 0: return tile_launch<256, 256, 2, 4, false>(a, e, x_hi, s);
    case 1: return tile_launch<128, 128, 4, 2, false>(a, e, x_hi, s);
    case 2: return tile_launch<128, 64, 2, 2, false>(a, e, x_hi, s);
    case 3: return tile_launch<64, 64, 2, 2, false>(a, e, x_hi, s);
    default: return tile_launch<64, 32, 2, 1, false>(a, e, x_hi, s);
    }
}

}  // namespace hawq
