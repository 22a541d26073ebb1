// Split-reduction implicit GEMM: the kernel for launches too small to fill the chip (and for a packed channel count that is a
// multiple of 16 only, and long packed reductions just above its line, at any size; conv_tile.hip takes the other large launches whose
// channel count no 64-channel K-step divides).
//
// Same GEMM view as conv_mfma.hip (rows = output channels, columns = output pixels, reduction index = (r, s, c)), another
// division of labour.  What bounds a small layer is latency: with few output tiles every workgroup walks its whole
// reduction step by step, and the tiled kernels pay a landing wait and a barrier per 64 reduction elements.  Here the
// WK waves of a workgroup *split the reduction* of one output tile, every wave requests all of its operands at once (or
// keeps a deep ring of them in flight), straight into registers, and the partial tiles meet once, in LDS (integer addition
// is associative: no bit changes).  No LDS and no barrier in the loop.
//
// The 16x16x64 MFMA makes that loading efficient: its operand fragment is 16 rows x 64 contiguous bytes, four lanes per
// row, which a CU's vector-memory path serves at its full ~60 B/clk (a 32x32x32 fragment, 32 rows x 32 bytes, gets a
// quarter of that).
//
// Each lane walks its own 16-byte chunk (FORM 2: 8-byte) of the flattened reduction index and finds its filter tap with two
// multiplications by a reciprocal, so a chunk only has to lie within one tap: C need only be a multiple of 16.
// FORM 0: 8-bit operands.  FORM 1: packed 4-bit, 16-byte chunks (C a multiple of 32), split into nibbles before two MFMAs.
// FORM 2: packed 4-bit, 8-byte chunks (C a multiple of 16), split into one 16-byte fragment.
// XF: unsigned bytes above 127 (hawq_gemm_int takes them): the kernel multiplies x XOR 0x80 = x - 128 and subtracts
// sum(w * -128), accumulated by one more MFMA per step against a constant operand; padding reads as -128 on both sides
// and cancels.
// A block output with two convolutions (ConvArgs::xs) divides the waves between them in proportion to their steps.
#include "common.h"
#include "fastdiv.h"

namespace hawq {

struct SkArgs {
    FastDiv ch, S, PQ, Q;      // 16-byte (8-byte) chunks of a tap, filter width, output pixels of an image, output width
    FastDiv ch_s;              // chunks of the shortcut convolution (one tap)
    int32_t wk_main;           // waves (of WK) on the main convolution; the others take the shortcut's
    uint32_t n_ct;             // channel tiles
    int32_t vec;               // K % 4 == 0 and aligned arrays: vector loads and stores in the epilogue
};

struct SkParams { int32_t bias[4], b[4], rb[4]; uint32_t c, rc, res; int32_t bias_s[4], b_s[4]; uint32_t c_s; };

// Shortcut values of channels ch .. ch + 3 at pixel m
__device__ __forceinline__ uint32_t sk_load_res(const ConvArgs &a, int vec, uint32_t m, int ch) {
    const int res_dt = a.res_dt;
    if (vec) {
        const uint32_t o = m * (uint32_t)a.K + ch;
        return is4(res_dt) ? *(const uint16_t *)(a.res + (o >> 1)) : *(const uint32_t *)(a.res + o);
    }
    uint32_t v = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int k = ch + j < a.K ? ch + j : a.K - 1;
        const int bits = is4(res_dt) ? 4 : 8;
        v |= ((uint32_t)load_elem(a.res, res_dt, (int64_t)m * a.K + k) & ((1u << bits) - 1)) << (bits * j);
    }
    return v;
}

// Parameters of channels ch .. ch + 3; RES: also the shortcut values at pixel m
template <bool DUAL, bool RES>
__device__ __forceinline__ void sk_load_params(const ConvArgs &a, int vec, uint32_t m, int ch, SkParams &p) {
    const bool rq = a.b != nullptr;
    if (RES && a.res != nullptr) p.res = sk_load_res(a, vec, m, ch);
    if (vec) {
        const v4i t = *(const v4i *)(a.bias + ch);
#pragma unroll
        for (int j = 0; j < 4; ++j) p.bias[j] = t[j];
        if (rq) {
            const v4i u = *(const v4i *)(a.b + ch);
#pragma unroll
            for (int j = 0; j < 4; ++j) p.b[j] = u[j];
            p.c = *(const uint32_t *)(a.c + ch);
        }
        if (a.res_b != nullptr) {
            const v4i u = *(const v4i *)(a.res_b + ch);
#pragma unroll
            for (int j = 0; j < 4; ++j) p.rb[j] = u[j];
            p.rc = *(const uint32_t *)(a.res_c + ch);
        }
        if constexpr (DUAL) {
            const v4i u = *(const v4i *)(a.bias_s + ch), v = *(const v4i *)(a.b_s + ch);
#pragma unroll
            for (int j = 0; j < 4; ++j) { p.bias_s[j] = u[j]; p.b_s[j] = v[j]; }
            p.c_s = *(const uint32_t *)(a.c_s + ch);
        }
    } else {
        p.c = p.rc = p.c_s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = ch + j < a.K ? ch + j : a.K - 1;
            p.bias[j] = a.bias[k];
            if (rq) { p.b[j] = a.b[k]; p.c |= (uint32_t)a.c[k] << (8 * j); }
            if (a.res_b != nullptr) { p.rb[j] = a.res_b[k]; p.rc |= (uint32_t)a.res_c[k] << (8 * j); }
            if constexpr (DUAL) { p.bias_s[j] = a.bias_s[k]; p.b_s[j] = a.b_s[k]; p.c_s |= (uint32_t)a.c_s[k] << (8 * j); }
        }
    }
}

// Four consecutive channels of one pixel: exact 64-bit evaluation (a thread has few outputs here), clamp, pack, store
template <bool DUAL>
__device__ __forceinline__ void sk_store(const ConvArgs &a, int vec, uint32_t m, int ch, v4i t, v4i ts, const SkParams &p) {
    const bool rq = a.b != nullptr, has_res = a.res != nullptr;
    const int y_dt = a.y_dt;
    int32_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int32_t u = t[j] + p.bias[j];
        if (!rq) { v[j] = u; continue; }
        int64_t y = rq64(u, p.b[j], (p.c >> (8 * j)) & 0xff);
        if (has_res) {
            int32_t r;
            if (is4(a.res_dt)) {
                r = (p.res >> (4 * j)) & 0xf;
                if (a.res_dt == HAWQ_S4) r = (r ^ 8) - 8;
            } else {
                r = (p.res >> (8 * j)) & 0xff;
                if (a.res_dt == HAWQ_S8) r = (int32_t)(int8_t)r;
            }
            y += rq64(r, p.rb[j], (p.rc >> (8 * j)) & 0xff);
        }
        if constexpr (DUAL) {
            int64_t s = rq64(ts[j] + p.bias_s[j], p.b_s[j], (p.c_s >> (8 * j)) & 0xff);
            if (a.mid_s8) s = rq64(clamp64(s, -128, 127), p.rb[j], (p.rc >> (8 * j)) & 0xff);
            y += s;
        }
        v[j] = clamp64(y, a.lo, a.hi);
    }
    const uint32_t o = m * (uint32_t)a.K + ch;
    if (vec) {
        if (y_dt == HAWQ_S32) *(v4i *)(a.y + 4 * (size_t)o) = (v4i){v[0], v[1], v[2], v[3]};
        else if (is4(y_dt)) *(uint16_t *)(a.y + (o >> 1)) = (uint16_t)((v[0] & 0xf) | ((v[1] & 0xf) << 4) | ((v[2] & 0xf) << 8) | ((v[3] & 0xf) << 12));
        else *(uint32_t *)(a.y + o) = (v[0] & 0xff) | ((v[1] & 0xff) << 8) | ((v[2] & 0xff) << 16) | ((uint32_t)v[3] << 24);
        return;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (ch + j >= a.K) continue;
        if (y_dt == HAWQ_S32) ((int32_t *)a.y)[o + j] = v[j];
        else if (!is4(y_dt)) a.y[o + j] = (uint8_t)v[j];
        else if ((j & 1) == 0) a.y[(o + j) >> 1] = (uint8_t)((v[j] & 0xf) | ((v[j + 1] & 0xf) << 4));   // (K is even)
    }
}

// A wave's tile: 16 TC channels x 16 TP pixels.  WK waves share it along the reduction, WM tiles lie side by side along the
// pixels of a workgroup.
template <int TC, int TP, int WK, int WM, int FORM, bool XF, bool DUAL>
__global__ void __launch_bounds__(WK *WM * 64) conv_sk_kernel(const ConvArgs a, const SkArgs e) {
    constexpr int CB = FORM == 2 ? 8 : 16;                  // bytes of a chunk
    constexpr int D = TC + TP <= 2 ? 8 : TC + TP <= 4 ? 5 : TC + TP <= 6 ? 4 : 3;   // steps in flight per wave
    constexpr int SLOTS = WM * TC * TP * 64, NT = WK * WM * 64, E = (SLOTS + NT - 1) / NT;
    constexpr uint32_t kInvalid = 0x80000000u;              // beyond every tensor: the load returns zeros
    static_assert(WK > 1, "the partial tiles meet in LDS, and two convolutions need two waves");
    __shared__ v4i red[WM * WK * TC * TP * 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % WK, wp = wave / WK;
    const int row16 = lane & 15, kg = lane >> 4;
    const uint32_t ct = blockIdx.x % e.n_ct, mt = blockIdx.x / e.n_ct;
    const int k0 = (int)ct * 16 * TC;
    const uint32_t m0 = mt * (16 * TP * WM);

    // ---- this wave's convolution and its share of the steps ----
    const bool on_s = DUAL && wk >= e.wk_main;
    const uint8_t *xp = on_s ? a.xs : a.x;
    const int H = on_s ? a.Hs : a.H, W = on_s ? a.Ws : a.W, C = on_s ? a.Cs : a.C;
    const int Cb = FORM == 0 ? C : C / 2;
    const int taps = on_s ? 1 : a.R * a.S;
    const int sh = on_s ? a.stride_sh : a.stride_h, sw = on_s ? a.stride_sw : a.stride_w;
    const int ph = on_s ? 0 : a.pad_h, pw = on_s ? 0 : a.pad_w;
    const FastDiv dch = on_s ? e.ch_s : e.ch;
    const int n_ch = Cb / CB, n_chunks = taps * n_ch, steps = (n_chunks + 3) >> 2;
    const int first = on_s ? wk - e.wk_main : wk, stride = !DUAL ? WK : on_s ? WK - e.wk_main : e.wk_main;
    const int n = first < steps ? (steps - first + stride - 1) / stride : 0;
    // weights: [K][row], or -- every K-step a whole 64-byte block -- the blocked copy (see ConvArgs::w_t)
    const void *wt = on_s ? a.ws_t : a.w_t;
    const bool tiled = FORM != 2 && wt != nullptr;
    const int row = taps * Cb;
    const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc((void *)(tiled ? wt : on_s ? a.ws : a.w), 0,
                                                                          tiled ? (a.K + 63) / 64 * steps * 4096 : a.K * row, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void *)xp, 0, a.N * H * W * Cb, 0x00020000);
    uint32_t woff[TC];
    const uint32_t wstep = tiled ? 4096 : 4 * CB;
#pragma unroll
    for (int tc = 0; tc < TC; ++tc) {
        const int k = k0 + tc * 16 + row16;
        woff[tc] = k >= a.K ? kInvalid : tiled ? (uint32_t)((k >> 6) * steps * 4096 + (k & 63) * 64 + kg * 16) : (uint32_t)(k * row + kg * CB);
    }
    uint32_t xoff[TP];
    int ih0[TP], iw0[TP];
#pragma unroll
    for (int tp = 0; tp < TP; ++tp) {
        const uint32_t m = m0 + (wp * TP + tp) * 16 + row16;
        const uint32_t nn = fdiv(m, e.PQ), pq = m - nn * (uint32_t)(a.P * a.Q);
        const uint32_t p = fdiv(pq, e.Q), q = pq - p * (uint32_t)a.Q;
        ih0[tp] = (int)p * sh - ph;
        iw0[tp] = (int)q * sw - pw;
        xoff[tp] = (uint32_t)((((int)nn * H + ih0[tp]) * W + iw0[tp]) * Cb);
        if (m >= (uint32_t)a.M) ih0[tp] = 1 << 30;          // (fails the bounds test of every tap)
    }
    // ---- parameters and shortcut values of the outputs this thread will finish: requested before the operands.  Of more than
    // two slots only the parameters, once: the slots lie whole rows of channel tiles apart and share them (loaded again for each
    // slot they cannot pass the stores before them: 39200 pixels of 1x1 288 -> 64 17.1 us, once 13.0) ----
    static_assert(E <= 2 || NT / 64 % TC == 0, "one set of channels per thread");
    SkParams par[E <= 2 ? E : 1];
    auto slot_mk = [&](int s, uint32_t &m, int &ch) {       // slot -> pixel, first of four channels
        const int l = s & 63, t = (s >> 6) % (TC * TP), w = s / (64 * TC * TP);
        m = m0 + (w * TP + t / TC) * 16 + (l & 15);
        ch = k0 + (t % TC) * 16 + (l >> 4) * 4;
    };
    if constexpr (E <= 2) {
#pragma unroll
        for (int j = 0; j < E; ++j) {
            uint32_t m; int ch;
            slot_mk(tid + j * NT, m, ch);
            if ((SLOTS % NT == 0 || tid + j * NT < SLOTS) && m < (uint32_t)a.M && ch < a.K) sk_load_params<DUAL, true>(a, e.vec, m, ch, par[j]);
        }
    } else {
        uint32_t m; int ch;
        slot_mk(tid, m, ch);
        if (ch < a.K) sk_load_params<DUAL, false>(a, e.vec, m, ch, par[0]);
    }

    v4i acc[TP][TC], accx[XF ? TC : 1];
#pragma unroll
    for (int tc = 0; tc < TC; ++tc) {
#pragma unroll
        for (int tp = 0; tp < TP; ++tp) acc[tp][tc] = (v4i){0, 0, 0, 0};
        if constexpr (XF) accx[tc] = (v4i){0, 0, 0, 0};
    }
    v4i fa[D][TC], fb[D][TP];
    auto load = [&](int i, v4i(&ra)[TC], v4i(&rb)[TP]) {    // the wave's i-th step
        const int step = first + i * stride;
        const uint32_t chunk = step * 4 + kg;
        const uint32_t tap = fdiv(chunk, dch), cc = chunk - tap * n_ch;
        const uint32_t r = on_s ? 0 : fdiv(tap, e.S), s = on_s ? 0 : tap - r * (uint32_t)a.S;
        const uint32_t off = (r * W + s) * Cb + cc * CB;
        const bool in = chunk < (uint32_t)n_chunks;
#pragma unroll
        for (int tc = 0; tc < TC; ++tc) {
            if constexpr (FORM == 2) {
                const v2i t = __builtin_amdgcn_raw_buffer_load_b64(rs_w, (int)(woff[tc] + step * wstep), 0, 0);
                ra[tc][0] = t[0]; ra[tc][1] = t[1];
            } else {
                ra[tc] = __builtin_amdgcn_raw_buffer_load_b128(rs_w, (int)(woff[tc] + step * wstep), 0, 0);
            }
        }
#pragma unroll
        for (int tp = 0; tp < TP; ++tp) {
            const bool ok = in & ((uint32_t)(ih0[tp] + (int)r) < (uint32_t)H) & ((uint32_t)(iw0[tp] + (int)s) < (uint32_t)W);
            const int o = (int)(ok ? xoff[tp] + off : kInvalid);
            if constexpr (FORM == 2) {
                const v2i t = __builtin_amdgcn_raw_buffer_load_b64(rs_x, o, 0, 0);
                rb[tp][0] = t[0]; rb[tp][1] = t[1];
            } else {
                rb[tp] = __builtin_amdgcn_raw_buffer_load_b128(rs_x, o, 0, 0);
            }
        }
    };
    // 4-bit fragments: activations become bytes 0..15, weights stay in the upper half of their byte (16 w, sign in place);
    // the sums are shifted back once at the end
    auto mul = [&](const v4i(&ra)[TC], const v4i(&rb)[TP]) {
        if constexpr (FORM == 0) {
            v4i b[TP];
#pragma unroll
            for (int tp = 0; tp < TP; ++tp) b[tp] = XF ? rb[tp] ^ (int)0x80808080 : rb[tp];
#pragma unroll
            for (int tc = 0; tc < TC; ++tc) {
#pragma unroll
                for (int tp = 0; tp < TP; ++tp) acc[tp][tc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ra[tc], b[tp], acc[tp][tc], 0, 0, 0);
                if constexpr (XF) {
                    const int c = (int)0x80808080;
                    accx[tc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ra[tc], (v4i){c, c, c, c}, accx[tc], 0, 0, 0);
                }
            }
        } else if constexpr (FORM == 1) {
            v4i bl[TP], bh[TP];
#pragma unroll
            for (int tp = 0; tp < TP; ++tp) { bl[tp] = rb[tp] & 0x0F0F0F0F; bh[tp] = (rb[tp] >> 4) & 0x0F0F0F0F; }
#pragma unroll
            for (int tc = 0; tc < TC; ++tc) {
                const v4i al = (ra[tc] << 4) & (int)0xF0F0F0F0, ah = ra[tc] & (int)0xF0F0F0F0;
#pragma unroll
                for (int tp = 0; tp < TP; ++tp) {
                    acc[tp][tc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(al, bl[tp], acc[tp][tc], 0, 0, 0);
                    acc[tp][tc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ah, bh[tp], acc[tp][tc], 0, 0, 0);
                }
            }
        } else {
            v4i b[TP];
#pragma unroll
            for (int tp = 0; tp < TP; ++tp)
                b[tp] = (v4i){rb[tp][0] & 0x0F0F0F0F, rb[tp][1] & 0x0F0F0F0F, (rb[tp][0] >> 4) & 0x0F0F0F0F, (rb[tp][1] >> 4) & 0x0F0F0F0F};
#pragma unroll
            for (int tc = 0; tc < TC; ++tc) {
                const int m = (int)0xF0F0F0F0;
                const v4i w = {(ra[tc][0] << 4) & m, (ra[tc][1] << 4) & m, ra[tc][0] & m, ra[tc][1] & m};
#pragma unroll
                for (int tp = 0; tp < TP; ++tp) acc[tp][tc] = __builtin_amdgcn_mfma_i32_16x16x64_i8(w, b[tp], acc[tp][tc], 0, 0, 0);
            }
        }
    };
    if (n <= D) {           // everything in flight at once
        static_for<0, D>([&](auto d) { if (decltype(d)::value < n) load(decltype(d)::value, fa[decltype(d)::value], fb[decltype(d)::value]); });
        static_for<0, D>([&](auto d) { if (decltype(d)::value < n) mul(fa[decltype(d)::value], fb[decltype(d)::value]); });
    } else {                // a ring of D steps; the last round refills only what is left
        static_for<0, D>([&](auto d) { load(decltype(d)::value, fa[decltype(d)::value], fb[decltype(d)::value]); });
        int i = D;
        for (; i + D <= n; i += D)
            static_for<0, D>([&](auto d) {
                constexpr int j = decltype(d)::value;
                mul(fa[j], fb[j]);
                load(i + j, fa[j], fb[j]);
            });
        const int rem = n - i;
        static_for<0, D>([&](auto d) {
            constexpr int j = decltype(d)::value;
            mul(fa[j], fb[j]);
            if (j < rem) load(i + j, fa[j], fb[j]);
        });
        static_for<0, D - 1>([&](auto d) { if (decltype(d)::value < rem) mul(fa[decltype(d)::value], fb[decltype(d)::value]); });
    }
#pragma unroll
    for (int tc = 0; tc < TC; ++tc)
#pragma unroll
        for (int tp = 0; tp < TP; ++tp) {
            if constexpr (XF) acc[tp][tc] -= accx[tc];
            if constexpr (FORM != 0) acc[tp][tc] >>= 4;
        }

    // ---- the partial tiles meet; every thread finishes four channels of a pixel ----
#pragma unroll
    for (int tp = 0; tp < TP; ++tp)
#pragma unroll
        for (int tc = 0; tc < TC; ++tc) red[((wp * WK + wk) * TC * TP + tp * TC + tc) * 64 + lane] = acc[tp][tc];
    __syncthreads();
    static_for<0, E>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const int s = tid + j * NT;
        if (SLOTS % NT != 0 && s >= SLOTS) return;
        uint32_t m; int ch;
        slot_mk(s, m, ch);
        if (m >= (uint32_t)a.M || ch >= a.K) return;
        v4i t = {0, 0, 0, 0}, ts = {0, 0, 0, 0};
        const int w = s / (64 * TC * TP), in_tile = s % (64 * TC * TP);
#pragma unroll
        for (int k = 0; k < WK; ++k) {
            const v4i u = red[(w * WK + k) * (64 * TC * TP) + in_tile];
            if (!DUAL || k < e.wk_main) t += u; else ts += u;
        }
        if constexpr (E <= 2) {
            sk_store<DUAL>(a, e.vec, m, ch, t, ts, par[j]);
        } else {
            if (a.res != nullptr) par[0].res = sk_load_res(a, e.vec, m, ch);
            sk_store<DUAL>(a, e.vec, m, ch, t, ts, par[0]);
        }
    });
}

// ---- host side ----

static int sk_form(const ConvArgs &a) { return !is4(a.x_dt) ? 0 : a.C % 32 == 0 ? 1 : 2; }

bool conv_sk_eligible(const ConvArgs &a) {
    const bool four = is4(a.x_dt);
    if (a.C % 16 != 0 || four != is4(a.w_dt)) return false;
    if (four ? (a.x_dt != HAWQ_U4 || a.w_dt != HAWQ_S4) : (a.w_dt != HAWQ_S8 || (a.x_dt != HAWQ_U8 && a.x_dt != HAWQ_S8))) return false;
    if (((uintptr_t)a.x | (uintptr_t)a.w) & 15) return false;
    const int64_t red = (int64_t)a.R * a.S * a.C;
    // packed sums are kept times sixteen: |16 w x| <= 16 * 8 * 15 and red < 2^20 stay below 2^31; the spatial limits are the bounds test's
    if (red >= (four ? 1 << 20 : 1 << 23) || (int64_t)a.H + a.R >= (1 << 29) || (int64_t)a.W + a.S >= (1 << 29)) return false;
    if ((int64_t)((a.K + 63) / 64 * 64) * (red + 64) >= ((int64_t)1 << 31)) return false;   // the blocked copy below the out-of-range offset
    return a.xs == nullptr;
}

bool conv_sk_dual_eligible(const ConvArgs &a, int x_hi, int xs_hi) {
    if (a.xs == nullptr || a.res != nullptr || a.b == nullptr || a.b_s == nullptr) return false;
    if (a.mid_s8 && (a.res_b == nullptr || a.res_c == nullptr)) return false;
    ConvArgs m = a;
    m.xs = nullptr;
    if (!conv_sk_eligible(m) || is4(a.x_dt) || is4(a.xs_dt) || a.Cs % 16 != 0 || a.ws_dt != HAWQ_S8) return false;
    if ((a.x_dt == HAWQ_U8 && x_hi > 127) || (a.xs_dt == HAWQ_U8 && xs_hi > 127)) return false;
    if (((uintptr_t)a.xs | (uintptr_t)a.ws) & 15) return false;
    return (int64_t)a.Hs < (1 << 29) && (int64_t)a.Ws < (1 << 29) && (int64_t)((a.K + 63) / 64 * 64) * (a.Cs + 64) < ((int64_t)1 << 31);
}

template <int TC, int TP, int WK, int WM>
static hawq_status sk_launch(const ConvArgs &a, SkArgs e, bool xf, hipStream_t s) {
    e.n_ct = (a.K + 16 * TC - 1) / (16 * TC);
    const uint32_t n_mt = (a.M + 16 * TP * WM - 1) / (16 * TP * WM), nb = e.n_ct * n_mt;
    constexpr int T = WK * WM * 64;
    e.wk_main = WK;
    if (a.xs != nullptr) {
        const int s1 = a.R * a.S * (a.C / 16), s2 = a.Cs / 16;
        const int w2 = (2 * WK * s2 + s1 + s2) / (2 * (s1 + s2));
        e.wk_main = WK - (w2 < 1 ? 1 : w2 > WK - 1 ? WK - 1 : w2);
        conv_sk_kernel<TC, TP, WK, WM, 0, false, true><<<nb, T, 0, s>>>(a, e);
        return check_launch();
    }
    const int form = sk_form(a);
    if (form == 1) conv_sk_kernel<TC, TP, WK, WM, 1, false, false><<<nb, T, 0, s>>>(a, e);
    else if (form == 2) conv_sk_kernel<TC, TP, WK, WM, 2, false, false><<<nb, T, 0, s>>>(a, e);
    else if (xf) conv_sk_kernel<TC, TP, WK, WM, 0, true, false><<<nb, T, 0, s>>>(a, e);
    else conv_sk_kernel<TC, TP, WK, WM, 0, false, false><<<nb, T, 0, s>>>(a, e);
    return check_launch();
}

// Launches this kernel is preferred for although a tiled or resident-pixel kernel takes the shape: up to 2^19 outputs, i.e.
// at most 256 tiles of 32 x 64.  Measured on the ResNet layers in both operand widths (weights not in L2, this kernel
// against the one it replaces): 7x7 3x3 512 -> 512 at batch 1 / 4 5.2 / 7.2 us (14.6 / 15.2), 14x14 3x3 256 -> 256 4.2 / 6.3
// (9.4 / 9.7), 28x28 3x3 128 -> 128 4.1 / 6.2 (7.1 / 8.6), 14x14 1x1 1024 -> 256 3.7 / 4.8 (8.7 / 9.0).  Above the line the
// streaming and resident-pixel kernels win: 56x56 1x1 64 -> 256 + shortcut at batch 4 16.3 (6.1), 28x28 128 -> 512 9.5 (6.5).
// One kind above 2^18 outputs is the tiled kernel's: a long 8-bit reduction over fewer than 1024 pixels, where that one takes 64 x 64
// tiles with a ring of eight -- unless the blocked copy of the weights, which both read, is there (without it, 7x7 2048 -> 512 at
// batch 16 9.7 us here, 8.6 there; 14x14 1024 -> 512 at 4 7.6 and 6.9; 128 x 4096 -> 4096 14.8 and 13.5).  Others are conv_tile.hip's
// (conv_tile_over_sk).
bool conv_sk_small(const ConvArgs &a) {
    const int64_t out = (int64_t)a.M * a.K;
    const bool tiled = !is4(a.x_dt) && a.xs == nullptr && a.w_t == nullptr && a.M < 1024 && (int64_t)a.R * a.S * a.C >= 1024 && a.C % 64 == 0 && a.K % 16 == 0;
    return out <= (tiled ? 1 << 18 : 1 << 19);
}

hawq_status launch_conv_sk(const ConvArgs &a_in, int x_hi, hipStream_t s) {
    ConvArgs a = a_in;
    if (a.M == 0) return HAWQ_OK;
    const int cb = sk_form(a) == 2 ? 8 : 16;
    SkArgs e{};
    e.ch = fast_div((is4(a.x_dt) ? a.C / 2 : a.C) / cb);
    e.S = fast_div(a.S);
    e.PQ = fast_div(a.P * a.Q);
    e.Q = fast_div(a.Q);
    e.ch_s = fast_div(a.xs != nullptr ? a.Cs / 16 : 1);
    // the blocked copy holds whole 64-byte K-steps of one tap each
    if (a.C % (is4(a.x_dt) ? 128 : 64) != 0) a.w_t = nullptr;
    if (a.xs != nullptr && a.Cs % 64 != 0) a.ws_t = nullptr;
    uintptr_t al = (uintptr_t)a.bias | (uintptr_t)a.b | (uintptr_t)a.res_b | (uintptr_t)a.bias_s | (uintptr_t)a.b_s;
    al |= (((uintptr_t)a.c | (uintptr_t)a.res_c | (uintptr_t)a.c_s) & 3) | (a.y_dt == HAWQ_S32 ? (uintptr_t)a.y : (uintptr_t)a.y & 3) | ((uintptr_t)a.res & 3);
    e.vec = a.K % 4 == 0 && (al & 15) == 0;
    const bool xf = a.x_dt == HAWQ_U8 && x_hi > 127;
    // The smallest tile whose workgroups still fit one round of 256 CUs: fewer, larger tiles leave CUs idle, and a CU draws
    // ~57 KB/us of operands from behind its L2 however large the tile is; a second round costs a whole workgroup life
    // (~1.6 us) more.  7x7 3x3 512 -> 512 at batch 1: 16x16 tiles (128 workgroups) 5.2 us, 32x32 (32) 8.0; 14x14 3x3
    // 256 -> 256 at batch 4: 32x32 (200) 6.3, 16x32 (400) 7.9, 16x16 (784) 9.1.  A 32x64 tile of few steps splits them
    // over four waves instead of eight (28x28 1x1 512 -> 128 at batch 4: 4.9 against 5.1 us), one of many over eight (7x7
    // 3x3 at batch 16: 12.4 against 13.9).  Past one round the number of waves in flight counts more than the operand bytes:
    // four waves a tile for long reductions (64 x 64; packed 5x5 240 -> 208 at 3267 pixels 22.4 us, with two 26.0), else two, 32 channels x
    // 64 pixels a workgroup, from 512 of those on 32 x 128 (packed 1x1 272 -> 288 at 39200 pixels 24 us,
    // with 64 x 128 tiles or four waves a tile 27 to 42; packed 3x3 48 -> 64 8.3 and 9.8) -- of more than 32 channels in their last 64,
    // between one round of the small tiles and two, only reductions of a few steps (1x1 544 -> 36 at 12887 pixels with a shortcut 5.6 us, in small
    // tiles 6.7; 3x3 96 -> 42 at 11025 6.7 and 7.6; with up to 4 steps, packed 6, the small ones are the faster or equal) and
    // two convolutions always (56 x 56, 160 -> 256 plus 1024 / 2 8.9 us, in small tiles 10.9; 32 x 32, 64 -> 756 plus 1024 / 2 10.6 and 11.9).
    auto tiles = [&](int tc, int tp) { return (int64_t)((a.K + 16 * tc - 1) / (16 * tc)) * ((a.M + 16 * tp - 1) / (16 * tp)); };
    if (tiles(1, 1) <= 256) return sk_launch<1, 1, 8, 1>(a, e, xf, s);
    if (tiles(1, 2) <= 256) return sk_launch<1, 2, 8, 1>(a, e, xf, s);
    if (tiles(2, 2) <= 256) return sk_launch<2, 2, 8, 1>(a, e, xf, s);
    const int steps = (a.R * a.S * (is4(a.x_dt) ? a.C / 2 : a.C) + 63) / 64;
    if (tiles(2, 4) <= 256) return steps < 32 ? sk_launch<2, 2, 4, 2>(a, e, xf, s) : sk_launch<2, 4, 8, 1>(a, e, xf, s);
    const bool whole = (a.K - 1) % 64 >= 32 && tiles(2, 4) > 272 && tiles(2, 4) <= 512 && steps >= (is4(a.x_dt) ? 7 : 5);
    if (tiles(4, 4) <= 512 && (steps >= 16 || whole || a.xs)) return sk_launch<4, 2, 4, 2>(a, e, xf, s);
    return tiles(2, 4) <= 512 ? sk_launch<2, 2, 2, 2>(a, e, xf, s) : sk_launch<2, 4, 2, 2>(a, e, xf, s);
}

}  // namespace hawq
