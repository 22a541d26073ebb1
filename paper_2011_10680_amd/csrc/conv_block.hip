// A whole bottleneck block at 64 channels as one launch (ResNet50 stage 1): 1x1 to 64 channels, 3x3, 1x1 to 256 channels plus
// the shortcut -- the block's input itself or a 1x1 convolution of it (Figure 2, Section 3.3).
//
// As three launches these blocks move the input twice and both tensors in between, and each launch has a ramp-up and a tail:
// 56 x 56 at batch 128 91 to 94 us with an identity shortcut, 81 us at the transition, of which input and output (206 and 128 MB)
// need 40 and 25.  Here a workgroup walks over tiles of 14 x 8 output pixels; a tile's input with a border of one pixel, 16 x 10, comes
// to LDS once and serves as the first convolution's operand and as the shortcut, and what lies between the convolutions stays in
// LDS.  The first convolution is computed on the border too (160 pixels for 112).  64 and 61 us (kernel trace, in the network); HBM
// reads 105 MB for the identity block, each input byte once.  The vector pipe binds (half of all cycles at 256 rescaled outputs and
// as many shortcuts a pixel; the matrix pipe a quarter), with the barriers between the three parts.
//
// Four waves to a workgroup, two workgroups to a CU, so that one fetches and multiplies while the other requantises.  The weights
// of the second, third and shortcut convolutions live in registers, the first's in LDS (all in registers: 33 of them spilled at the
// transition, 86 us; the shortcut's in LDS too: no faster, and batch 128 as a whole 25 us slower).  The next tile's input comes
// while the second and third convolutions of this one run: the identity shortcut's bytes go to registers before, the transition's
// small input has two places in LDS.  Sixteen columns to a tile's input row make every LDS address of the kernel a lane's constant
// plus an immediate: pixel h of the input tile lies in row h, a tap's row distance is a multiple of sixteen rows and leaves the
// bank permutation as it is.
//
// Two waves a SIMD leave 256 registers, and not every form fits them: by the compiler's report the transition keeps 4 words a lane
// in scratch memory, with a stored shortcut 10, the identity block of bytes with integer shortcuts 6; in floating point and of
// packed 4-bit pixels none.  Batch 256: bytes 113 us, packed input 115, packed input and output 122, stored transition 132 (packed
// output 138).
//
// The identity shortcut of bytes is scaled in floating point, two instructions for three: 3.5 us of the identity block's 64,
// ResNet50 as a whole 966 -> 959 at batch 128.  (The streaming 1x1 kernels with a shortcut gained
// nothing by it: 32.3 us either way at 28 x 28, 21 at 14 x 14, batch 128.)
#include "conv_block.h"

namespace hawq {

namespace {

constexpr int TW = BLOCK_TW, TH = BLOCK_TH, HW16 = BLOCK_HW, HALO = HW16 * BLOCK_HROWS;   // 160 input pixels
constexpr uint32_t kOut = 0x80000000u;

__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// high word of t b + 2^31 (bias already in t): the narrow evaluation of rq
__device__ __forceinline__ int32_t scale(int32_t t, int32_t b, uint64_t r31) {
    return (int32_t)(((uint64_t)((int64_t)t * (int64_t)b) + r31) >> 32);
}
__device__ __forceinline__ int32_t med3(int32_t v, int32_t lo, int32_t hi) {
    int32_t o;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(o) : "v"(v), "v"(lo), "v"(hi));
    return o;
}
__device__ __forceinline__ v4i pack16(const int32_t (&y)[16]) {
    v4i o;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t t0 = __builtin_amdgcn_perm((uint32_t)y[4 * q + 1], (uint32_t)y[4 * q], 0x0c0c0400u);
        const uint32_t t1 = __builtin_amdgcn_perm((uint32_t)y[4 * q + 3], (uint32_t)y[4 * q + 2], 0x04000c0cu);
        o[q] = (int)(t0 | t1);
    }
    return o;
}
// kResMagic + the shortcut of byte I in floating point (conv_block_plan.h): two vector instructions, the conversion picks its byte
template <int I>
__device__ __forceinline__ int32_t res_term(uint32_t bytes, int32_t rf) {
    return res_scaled((float)((bytes >> (8 * I)) & 0xffu), rf);
}
// sixteen words of a lane's channels; fresh: read here, not kept from an earlier use (accumulators start at the bias, and a copy
// kept for all of them would be sixteen registers and sixteen moves for each)
template <bool FRESH = false>
__device__ __forceinline__ v16i words16(const int32_t *base, int at) {
    if (FRESH) asm volatile("" : "+v"(at));
    const int32_t *p = base + at;
    v16i v;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const v4i t = *(const v4i *)(p + 4 * q);
        v[4 * q] = t[0]; v[4 * q + 1] = t[1]; v[4 * q + 2] = t[2]; v[4 * q + 3] = t[3];
    }
    return v;
}

// DUAL: the shortcut is a 1x1 convolution of the input, which has 64 channels then, else 256; MID8: ... whose result passes through
// a signed byte; XPK / Y4: input / output packed 4-bit; FLT: the shortcut's bytes are scaled in floating point (res_float)
template <bool DUAL, bool MID8, bool XPK, bool Y4, bool FLT>
__global__ void __launch_bounds__(256, 2) block64_kernel(const BlockArgs a) {
    static_assert(!(DUAL && XPK) && !(FLT && (DUAL || XPK)), "the transition block's input has bytes; floating point is for bytes");
    constexpr int XB = DUAL ? 64 : XPK ? 128 : 256;          // bytes of an input pixel
    constexpr int P1 = DUAL ? 2 : 8;                         // 32-element pieces of the first convolution's reduction
    constexpr int NX = HALO * XB / 1024;                     // LDS-DMA instructions of a tile
    constexpr int PPI = 1024 / XB;                           // pixels of one
    constexpr int NPAR = DUAL ? 1536 : 1024;
    __shared__ __attribute__((aligned(1024))) uint8_t xs[(DUAL ? 2 : 1) * HALO * XB];   // (the small input: two tiles in turn)
    __shared__ __attribute__((aligned(1024))) uint8_t hs[HALO * 64];     // first convolution's results
    __shared__ __attribute__((aligned(1024))) uint8_t gs[128 * 64];      // second's
    __shared__ __attribute__((aligned(1024))) uint8_t ws[2 * P1 * 1024]; // first convolution's weights
    __shared__ __attribute__((aligned(16))) int32_t par[NPAR];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rho = lane & 31, kh = lane >> 5;
    const int rt = wave & 1, side = wave >> 1;               // channel half, pixel half of the first two convolutions

    for (int i = tid; i < NPAR / 4; i += 256) ((v4i *)par)[i] = ((const v4i *)a.par)[i];
    for (int i = tid; i < 2 * P1 * 64; i += 256) ((v4i *)ws)[i] = ((const v4i *)a.w1)[i];

    // ---- weights of the other convolutions ----
    v4i w2[18], w3[2][2], w4[DUAL ? 2 : 1][2];
    {
        const __amdgpu_buffer_rsrc_t r2 = __builtin_amdgcn_make_buffer_rsrc((void *)a.w2, 0, 36 * 1024, 0x00020000);
        const __amdgpu_buffer_rsrc_t r3 = __builtin_amdgcn_make_buffer_rsrc((void *)a.w3, 0, 16 * 1024, 0x00020000);
        const __amdgpu_buffer_rsrc_t r4 = __builtin_amdgcn_make_buffer_rsrc((void *)(DUAL ? a.w4 : a.w3), 0, 16 * 1024, 0x00020000);
#pragma unroll
        for (int i = 0; i < 18; ++i) w2[i] = __builtin_amdgcn_raw_buffer_load_b128(r2, lane * 16, (rt * 18 + i) * 1024, 0);
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                w3[j][i] = __builtin_amdgcn_raw_buffer_load_b128(r3, lane * 16, ((2 * wave + j) * 2 + i) * 1024, 0);
                if constexpr (DUAL) w4[j][i] = __builtin_amdgcn_raw_buffer_load_b128(r4, lane * 16, ((2 * wave + j) * 2 + i) * 1024, 0);
            }
    }
    // ---- a lane's constants ----
    // rows of XB bytes, the 16-byte chunks permuted by the row (modulo sixteen rows, which is what a column tile advances by)
    auto xswz = [](int h) { return DUAL ? (h >> 2) & 3 : XPK ? (h >> 1) & 7 : h & 15; };
    const uint32_t a1 = (uint32_t)(rho * XB + (((XPK ? 0 : kh) ^ xswz(rho)) << 4));      // first convolution: piece 0 of input pixel rho
    const uint32_t o1 = (uint32_t)(rho * 64 + (((2 * rt + kh) ^ ((rho >> 2) & 3)) << 4));   // its result; likewise the second's
    uint32_t a2[2][3];                                       // second convolution: column dc of the taps under pixel m, piece 0
    uint32_t px[4], ax[4];                                   // output pixel m: its place in the tile, its input pixel's chunk
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
        const int m = ct * 32 + rho, mm = min(m, TW * TH - 1), r = mm / TW, c = mm - r * TW;
        px[ct] = m < TW * TH ? (uint32_t)((r << 8) | c) : (uint32_t)(0xff << 8);      // (a row that no image reaches)
        const int h = (r + 1) * HW16 + c + 1;
        ax[ct] = (uint32_t)(h * XB + (XPK ? ((xswz(h) << 4) | (kh << 3)) : ((kh ^ xswz(h)) << 4)));
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int m = min((2 * side + j) * 32 + rho, TW * TH - 1), r = m / TW, c = m - r * TW;
#pragma unroll
        for (int dc = 0; dc < 3; ++dc) {
            const int h = r * HW16 + c + dc;
            a2[j][dc] = (uint32_t)(h * 64 + ((kh ^ ((h >> 2) & 3)) << 4));
        }
    }
    const uint32_t a3 = (uint32_t)(rho * 64 + ((kh ^ ((rho >> 2) & 3)) << 4));           // last convolution: piece 0 of pixel rho
    uint32_t r31 = 0x80000000u;                              // (opaque: with the constant in sight the multiply-add falls apart)
    uint64_t r3 = r31;                                       // the last convolution's: takes the shortcut's offset off again
    if constexpr (FLT) { r3 -= (uint64_t)kResMagic << 32; asm volatile("" : "+v"(r3)); }
    int32_t lo3 = a.lo3, hi1 = a.hi1, hi2 = a.hi2, hi3 = a.hi3, zero = 0;
    asm volatile("" : "+v"(r31), "+v"(lo3), "+v"(hi1), "+v"(hi2), "+v"(hi3), "+v"(zero));
    const int32_t T = a.t, half = (int32_t)(1u << (T - 1));

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void *)a.x, 0, (int)((int64_t)a.N * a.H * a.W * XB), 0x00020000);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void *)a.y, 0, (int)(((int64_t)a.N * a.H * a.W * 256) >> (Y4 ? 1 : 0)), 0x00020000);
    const TileWalk walk = xcd_walk(blockIdx.x, gridDim.x, a.n_tiles);
    const int per_image = a.tiles_x * a.tiles_y;

    int buf = 0;                                             // DUAL: which of the two the tile in work has
    auto fetch = [&](int tile, int to) {
        const int n = tile / per_image, t = tile - n * per_image, ty = t / a.tiles_x;
        const int y0 = ty * TH - 1, x0 = (t - ty * a.tiles_x) * TW - 1;
        constexpr int CPP = XB / 16, IPR = HW16 / PPI;       // chunks of a pixel, instructions of an input row
        const int hc = wave % IPR * PPI + lane / CPP, x = x0 + hc;       // (instruction 4 i + wave: part wave % IPR of a row)
        const uint32_t col = (unsigned)x < (unsigned)a.W ? (uint32_t)(x * XB + (((lane % CPP) ^ xswz(hc)) << 4)) : kOut;
#pragma unroll
        for (int i = 0; i < (NX + 3) / 4; ++i) {
            const int k = wave + 4 * i;
            if (NX % 4 != 0 && k >= NX) break;
            const int y = y0 + k / IPR;
            const uint32_t off = (unsigned)y < (unsigned)a.H ? col : kOut;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void *)(xs + to + k * 1024), 16, (int)off,
                                                     block_input_row(n, y, a.H, a.W, XB), 0, 0);
        }
    };

    int tile = walk.first;
    if (tile >= walk.end) return;                            // (the whole workgroup)
    fetch(tile, 0);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    for (;;) {
        const int n = tile / per_image, t = tile - n * per_image, ty = t / a.tiles_x;
        const int y0 = ty * TH, x0 = (t - ty * a.tiles_x) * TW;
        lds_barrier();                                       // the tile is here

        // ---- 1x1 to 64 channels, on the border too: five column tiles, three for one pair of waves and two for the other ----
        {
            v4i w1[P1];
#pragma unroll
            for (int i = 0; i < P1; ++i) w1[i] = *(const v4i *)(ws + (rt * P1 + i) * 1024 + lane * 16);
            const v16i b = words16(par, 64 + rt * 32 + kh * 16);
#pragma nounroll
            for (int ct = 3 * side; ct < 3 + 2 * side; ++ct) {
                v16i acc = words16<true>(par, rt * 32 + kh * 16);
                const uint8_t *base = xs + buf + ct * 32 * XB;
#pragma unroll
                for (int i = 0; i < P1; ++i) {
                    v4i v = *(const v4i *)(base + (a1 ^ (uint32_t)(i << (XPK ? 4 : 5))));
                    if constexpr (XPK) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = (int)(((uint32_t)v[e] >> (4 * kh)) & 0x0F0F0F0Fu);
                    }
                    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w1[i], v, acc, 0, 0, 0);
                }
                const int h = ct * 32 + rho, y = y0 - 1 + (h >> 4), x = x0 - 1 + (h & 15);
                const bool in = (unsigned)y < (unsigned)a.H && (unsigned)x < (unsigned)a.W;   // (the 3x3's padding is zeros)
                int32_t v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = med3(scale(acc[i], b[i], r31), zero, hi1);
                v4i o = pack16(v);
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = in ? o[i] : 0;
                *(v4i *)(hs + ct * 2048 + o1) = o;
            }
        }
        // the shortcut's bytes into registers: the tile's place is free for the next one
        v4i xr[DUAL ? 1 : 4][2];
        if constexpr (!DUAL)
#pragma unroll
            for (int ct = 0; ct < 4; ++ct)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    if constexpr (XPK) {
                        const v2i r = *(const v2i *)(xs + (ax[ct] ^ (uint32_t)((2 * wave + j) << 4)));
                        xr[ct][j] = (v4i){r[0], r[1], 0, 0};
                    } else xr[ct][j] = *(const v4i *)(xs + (ax[ct] ^ (uint32_t)((2 * wave + j) << 5)));
                }
        lds_barrier();
        const int next = tile + walk.step;
        const bool more = next < walk.end;
        if (more) fetch(next, DUAL ? HALO * XB - buf : 0);

        // ---- 3x3 ----
        {
            v16i acc[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[j] = words16<true>(par, 128 + rt * 32 + kh * 16);
#pragma unroll
            for (int i = 0; i < 18; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(w2[i], *(const v4i *)(hs + (a2[j][i / 2 % 3] ^ ((i & 1) << 5)) + (i / 6) * (HW16 * 64)), acc[j], 0, 0, 0);
            const v16i b = words16(par, 192 + rt * 32 + kh * 16);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                int32_t v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = med3(scale(acc[j][i], b[i], r31), zero, hi2);
                *(v4i *)(gs + (2 * side + j) * 2048 + o1) = pack16(v);
            }
        }
        lds_barrier();

        // ---- 1x1 to 256 channels, plus the shortcut ----
        uint32_t vo[4];                                      // where the lane's pixels go
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
            const int r = (int)(px[ct] >> 8), c = (int)(px[ct] & 0xff);
            vo[ct] = y0 + r < a.H && x0 + c < a.W && r < TH ? (uint32_t)((r * a.W + c) * 256 + kh * 16) >> (Y4 ? 1 : 0) : kOut;
        }
        const int first = (n * a.H + y0) * a.W + x0;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int ch = (2 * wave + j) * 32 + kh * 16;
            // (in the address, not in the instruction's scalar offset: behind a 128-bit store with a scalar offset the compiler lets
            // the next instruction overwrite the data, and with two waves on a SIMD that one came first)
            const uint32_t so = (uint32_t)(first * 256 + (2 * wave + j) * 32) >> (Y4 ? 1 : 0);
            const v16i b3 = words16(par, 512 + ch);
            v16i rb;
            if constexpr (!DUAL) rb = words16(par, 768 + ch);
#pragma unroll
            for (int ct = 0; ct < 4; ++ct) {
                v16i acc = words16<true>(par, 256 + ch);
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(w3[j][i], *(const v4i *)(gs + (a3 ^ (uint32_t)(i << 5)) + ct * 2048), acc, 0, 0, 0);
                int32_t v[16], z[16];
                if constexpr (DUAL) {
                    v16i acs = words16<true>(par, 1024 + ch);
#pragma unroll
                    for (int i = 0; i < 2; ++i) acs = __builtin_amdgcn_mfma_i32_32x32x32_i8(w4[j][i], *(const v4i *)(xs + buf + (ax[ct] ^ (uint32_t)(i << 5))), acs, 0, 0, 0);
                    const v16i b4 = words16<true>(par, 1280 + ch);
#pragma unroll
                    for (int i = 0; i < 16; ++i) z[i] = scale(acs[i], b4[i], r31);
                    if constexpr (MID8) {
                        const v16i q = words16<true>(par, 768 + ch);
#pragma unroll
                        for (int i = 0; i < 16; ++i) z[i] = (__mul24(min(max(z[i], -128), 127), q[i]) + half) >> T;
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        if constexpr (FLT) continue;
                        const uint32_t r = XPK ? __builtin_amdgcn_ubfe((uint32_t)xr[ct][j][i >> 3], 4 * (i & 7), 4)
                                               : __builtin_amdgcn_ubfe((uint32_t)xr[ct][j][i >> 2], 8 * (i & 3), 8);
                        z[i] = (__mul24((int)r, rb[i]) + half) >> T;
                    }
                    if constexpr (FLT)
                        static_for<0, 16>([&](auto ic) {
                            constexpr int i = decltype(ic)::value;
                            z[i] = res_term<(i & 3)>((uint32_t)xr[ct][j][i >> 2], rb[i]);
                        });
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = med3((int32_t)((uint32_t)scale(acc[i], b3[i], FLT ? r3 : r31) + (uint32_t)z[i]), lo3, hi3);
                const v4i o = pack16(v);
                if constexpr (Y4) {
                    auto nib = [](uint32_t d) { return (d & 0xfu) | ((d >> 4) & 0xf0u) | ((d >> 8) & 0xf00u) | ((d >> 12) & 0xf000u); };
                    __builtin_amdgcn_raw_buffer_store_b64((v2i){(int)(nib((uint32_t)o[0]) | (nib((uint32_t)o[1]) << 16)), (int)(nib((uint32_t)o[2]) | (nib((uint32_t)o[3]) << 16))},
                                                          ry, (int)(vo[ct] + so), 0, 0);
                } else {
                    __builtin_amdgcn_raw_buffer_store_b128(o, ry, (int)(vo[ct] + so), 0, 0);
                }
            }
        }
        if (!more) break;
        tile = next;
        if (DUAL) buf = HALO * XB - buf;
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");     // all but the eight stores behind it: the next tile
    }
}

}  // namespace

hawq_status launch_block64(const BlockArgs &args, hipStream_t s) {
    BlockArgs a = args;
    a.tiles_x = (a.W + TW - 1) / TW; a.tiles_y = (a.H + TH - 1) / TH;
    const int64_t n = (int64_t)a.N * a.tiles_x * a.tiles_y;
    if (n > 0x7fffffff || (int64_t)a.N * a.H * a.W * 256 >= 0x80000000ll) return HAWQ_ERR_UNSUPPORTED;
    if (n == 0) return HAWQ_OK;
    a.n_tiles = (int)n;
    const uint32_t grid = xcd_walk_grid(n, 2 * 256);
    auto go = [&](auto dual, auto mid8, auto xpk, auto flt) {
        if (a.y4) block64_kernel<decltype(dual)::value, decltype(mid8)::value, decltype(xpk)::value, true, decltype(flt)::value><<<grid, 256, 0, s>>>(a);
        else block64_kernel<decltype(dual)::value, decltype(mid8)::value, decltype(xpk)::value, false, decltype(flt)::value><<<grid, 256, 0, s>>>(a);
    };
    const std::true_type yes{};
    const std::false_type no{};
    if (a.w4 != nullptr && a.mid8) go(yes, yes, no, no);
    else if (a.w4 != nullptr) go(yes, no, no, no);
    else if (a.x4) go(no, no, yes, no);
    else if (a.flt) go(no, no, no, yes);
    else go(no, no, no, no);
    return check_launch();
}

}  // namespace hawq
