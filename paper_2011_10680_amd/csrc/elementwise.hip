// Memory-bound integer kernels: stand-alone dyadic residual add, global average pool,
// 3x3/2 max pool, INT32 window-sum pool, per-branch dyadic concatenation.  One thread handles 4 consecutive channels of one pixel when the channel
// count allows it (dword loads/stores of packed 8-bit data), else one unit of 1 or 2 channels.
#include "common.h"

namespace hawq {

// ---- residual add (Section 3.3): y = clamp(rq(m) + rq(r)) ----
__global__ void __launch_bounds__(256)
residual_add_kernel(const int64_t units, const int K, const int per, const int m_dt, const int r_dt, const int y_dt,
                    const void *m, const int32_t *__restrict__ m_b, const uint8_t *__restrict__ m_c,
                    const void *r, const int32_t *__restrict__ r_b, const uint8_t *__restrict__ r_c,
                    const int lo, const int hi, void *y) {   // (m, r, y unqualified: y may alias m or r when the types match)
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= units) return;
    const int64_t e0 = u * per;
    const int k0 = (int)(e0 % K);
    int32_t out[4];
    for (int j = 0; j < per; ++j) {
        const int k = k0 + j;
        const int64_t v = rq64(load_elem(m, m_dt, e0 + j), m_b[k], m_c[k]) + rq64(load_elem(r, r_dt, e0 + j), r_b[k], r_c[k]);
        out[j] = clamp64(v, lo, hi);
    }
    if (y_dt == HAWQ_S32) {
        for (int j = 0; j < per; ++j) ((int32_t *)y)[e0 + j] = out[j];
    } else if (is4(y_dt)) {
        for (int j = 0; j < per; j += 2) ((uint8_t *)y)[(e0 + j) >> 1] = (uint8_t)((out[j] & 0xf) | ((out[j + 1] & 0xf) << 4));
    } else if (per == 4) {
        ((uint32_t *)y)[e0 >> 2] = (out[0] & 0xff) | ((out[1] & 0xff) << 8) | ((out[2] & 0xff) << 16) | ((uint32_t)out[3] << 24);
    } else {
        for (int j = 0; j < per; ++j) ((uint8_t *)y)[e0 + j] = (uint8_t)out[j];
    }
}

// Vector form: K % 4 == 0, 8-bit or INT32 operands and output.  A thread keeps one group of four channels (the grid's thread
// count is a multiple of K / 4), so its parameters sit in registers, and has four pixels' loads in flight.  Bound: HBM
// (m, r and y once); 32 x 56 x 56 x 256 INT32 + u8 -> u8 (154 MB): 103 us in the element-wise form above, whose sixteen
// parameter loads per thread outnumbered its two data loads, 37 us (4.2 TB/s) in the exact 64-bit form below, 25.8 us (6.0 TB/s)
// in the streaming form after it.
template <int DT, bool NT = false>
__device__ __forceinline__ v4i load4(const void *p, int64_t unit) {   // elements 4 unit .. 4 unit + 3
    if constexpr (DT == HAWQ_S32) {
        if constexpr (NT) return __builtin_nontemporal_load((const v4i *)p + unit);
        else return ((const v4i *)p)[unit];
    } else {
        const uint32_t w = ((const uint32_t *)p)[unit];
        if constexpr (DT == HAWQ_U8) return (v4i){(int)(w & 0xff), (int)((w >> 8) & 0xff), (int)((w >> 16) & 0xff), (int)(w >> 24)};
        else return (v4i){(int)(int8_t)w, (int)(int8_t)(w >> 8), (int)(int8_t)(w >> 16), (int)w >> 24};
    }
}
template <int MD, int RD, bool Y32>
__global__ void __launch_bounds__(256)
residual_add_vec_kernel(const uint32_t units, const uint32_t groups, const void *m, const int32_t *__restrict__ m_b,
                        const uint8_t *__restrict__ m_c, const void *r, const int32_t *__restrict__ r_b,
                        const uint8_t *__restrict__ r_c, const int lo, const int hi, void *y) {
    constexpr int U = 4;
    const uint32_t T = gridDim.x * 256;
    uint32_t u = blockIdx.x * 256 + threadIdx.x;
    const uint32_t g = u % groups;
    const v4i mb = ((const v4i *)m_b)[g], rb = ((const v4i *)r_b)[g];
    const uint32_t mc = ((const uint32_t *)m_c)[g], rc = ((const uint32_t *)r_c)[g];
    auto finish = [&](const v4i &a, const v4i &b, uint32_t at) {
        v4i o;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            o[j] = clamp64(rq64(a[j], mb[j], (mc >> (8 * j)) & 0xff) + rq64(b[j], rb[j], (rc >> (8 * j)) & 0xff), lo, hi);
        if (Y32) ((v4i *)y)[at] = o;
        else ((uint32_t *)y)[at] = (o[0] & 0xff) | ((o[1] & 0xff) << 8) | ((o[2] & 0xff) << 16) | ((uint32_t)o[3] << 24);
    };
    for (; u + (U - 1) * T < units; u += U * T) {      // (units + U T stays far below 2^32: the interface takes fewer than 2^31 elements)
        v4i a[U], b[U];
#pragma unroll
        for (int i = 0; i < U; ++i) { a[i] = load4<MD>(m, u + i * T); b[i] = load4<RD>(r, u + i * T); }
#pragma unroll
        for (int i = 0; i < U; ++i) finish(a[i], b[i], u + i * T);
    }
    for (; u < units; u += T) {
        const v4i a = load4<MD>(m, u), b = load4<RD>(r, u);
        finish(a, b, u);
    }
}

// rq(t, b, c) of four channels whose parameters a thread keeps.  Narrow evaluation, exact like the 64-bit one, where the
// parameters allow it: INT32 operands (c <= 32, b < 2^(c-1)): high word of t * (b << (32 - c)) + 2^31, one instruction;
// 8-bit operands (c <= 31, b < 2^22): (t * b + 2^(c-1)) >> c in 32 bits, two.  Results then stay below 2^30, so two of them
// add up in 32 bits.  (The 64-bit form's shifts and comparisons, some 28 instructions per output of a residual addition, were
// 23 us of vector arithmetic next to 30 us of memory traffic in the case above; the narrow form's are 5.)
template <int DT>
struct Rescale4 {
    v4i b, k, rnd;     // k: b << (32 - c) (INT32) or c (8 bits)
    uint32_t c;
    __device__ __forceinline__ bool init(const v4i &b_, uint32_t c_) {
        b = b_; c = c_;
        bool ok = true;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t cj = (c >> (8 * j)) & 0xff;
            if constexpr (DT == HAWQ_S32) {
                ok &= cj <= 32 && ((uint32_t)b[j] >> ((cj - 1) & 31)) == 0;
                k[j] = (int32_t)((uint32_t)b[j] << ((32 - cj) & 31));
            } else {
                ok &= cj <= 31 && b[j] < (1 << 22);
                k[j] = (int32_t)(cj & 31);
                rnd[j] = (int32_t)(1u << ((cj - 1) & 31));
            }
        }
        return ok;
    }
    __device__ __forceinline__ int32_t narrow(int32_t t, int j, int64_t half) const {
        if constexpr (DT == HAWQ_S32) return (int32_t)(((int64_t)t * (int64_t)k[j] + half) >> 32);
        else return (__mul24(t, b[j]) + rnd[j]) >> k[j];
    }
    __device__ __forceinline__ int64_t wide(int32_t t, int j) const { return rq64(t, b[j], (c >> (8 * j)) & 0xff); }
};
__device__ __forceinline__ int32_t med3(int32_t v, int32_t lo, int32_t hi) {   // lo <= hi is validated by the interface
    int32_t t;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(t) : "v"(v), "v"(lo), "v"(hi));
    return t;
}
__device__ __forceinline__ uint32_t pack4(const v4i &o) {   // low bytes of four values
    return __builtin_amdgcn_perm((uint32_t)o[1], (uint32_t)o[0], 0x0c0c0400u) | __builtin_amdgcn_perm((uint32_t)o[3], (uint32_t)o[2], 0x04000c0cu);
}

// The form for tensors that many rounds of the grid stream through: narrow evaluation, three workgroups a compute unit.  NT: INT32
// operands pass the caches by (non-temporal loads).  Results do not: the layer that reads them next would find them in HBM (a
// convolution behind the addition 5 to 14 % slower over all sizes, 64 -> 512 at 236463 pixels 51 us for both, with non-temporal
// stores 75).
template <int MD, int RD, bool Y32, bool NT>
__global__ void __launch_bounds__(256)
residual_add_stream_kernel(const uint32_t units, const uint32_t groups, const void *m, const int32_t *__restrict__ m_b,
                        const uint8_t *__restrict__ m_c, const void *r, const int32_t *__restrict__ r_b,
                        const uint8_t *__restrict__ r_c, const int lo, const int hi, void *y) {
    constexpr int U = 4;
    const uint32_t T = gridDim.x * 256;
    uint32_t u = blockIdx.x * 256 + threadIdx.x;
    const uint32_t g = u % groups;
    const v4i mb = ((const v4i *)m_b)[g], rb = ((const v4i *)r_b)[g];
    const uint32_t mc = ((const uint32_t *)m_c)[g], rc = ((const uint32_t *)r_c)[g];
    v4i a[U], b[U];
    auto fetch = [&]() -> bool {       // four pixels' operands (units + U T stays far below 2^32: the interface takes fewer than 2^31 elements)
        const bool four = u + (U - 1) * T < units;
        if (four)
#pragma unroll
            for (int i = 0; i < U; ++i) { a[i] = load4<MD, NT>(m, u + i * T); b[i] = load4<RD, NT>(r, u + i * T); }
        return four;
    };
    bool four = fetch();               // (in flight while the parameters arrive and their form is decided)
    Rescale4<MD> pm;
    Rescale4<RD> pr;
    const bool ok_m = pm.init(mb, mc), narrow = pr.init(rb, rc) & ok_m;
    int32_t vlo = lo, vhi = hi;
    int64_t half = (int64_t)1 << 31;
    asm volatile("" : "+v"(vlo), "+v"(vhi), "+v"(half));   // (an addend that the compiler knows makes it split the multiply-add)
    auto walk = [&](auto nc) {
        auto finish = [&](const v4i &a, const v4i &b, uint32_t at) {
            v4i o;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (decltype(nc)::value) o[j] = med3(pm.narrow(a[j], j, half) + pr.narrow(b[j], j, half), vlo, vhi);
                else o[j] = clamp64(pm.wide(a[j], j) + pr.wide(b[j], j), lo, hi);
            }
            if (Y32) ((v4i *)y)[at] = o;
            else ((uint32_t *)y)[at] = pack4(o);
        };
        while (four) {
#pragma unroll
            for (int i = 0; i < U; ++i) finish(a[i], b[i], u + i * T);
            u += U * T;
            four = fetch();
        }
        for (; u < units; u += T) {
            const v4i a1 = load4<MD, NT>(m, u), b1 = load4<RD, NT>(r, u);
            finish(a1, b1, u);
        }
    };
    if (__all(narrow)) walk(std::true_type{});
    else walk(std::false_type{});
}

// Workgroups of 256 threads such that their threads are a multiple of `groups` (every thread keeps its channel group): a
// multiple of groups / gcd(groups, 256), one unit per thread up to `large` workgroups, which then walk.  0: no such grid.
// 1024 (four to a compute unit) and not one to each four units: that grid has its last round half empty (32 x 35 x 35 x 288 INT32 to
// 4 bits 11.1 us, with 1024 workgroups 10.2; four branches of 512 channels in all to 8 bits 19.9 and 18.7).
// stream: no more than `large` where a multiple at most an eighth below it exists, for a few compute units with one workgroup more than
// the others set the end (200704 pixels of 100 channels, INT32 and bytes, 775 workgroups 23.6 us, 750 21.2; 60000 of 300 21.7 and
// 19.6; 25088 of 1028 771 workgroups 29.2 us, 514 31.5).  The concatenation gains nothing from it (288 channels to 4 bits 10.7, 10.9).
static uint32_t grouped_blocks(int64_t units, uint32_t groups, int64_t large = 1024, bool stream = false) {
    uint32_t a = groups, b = 256;
    while (b) { const uint32_t t = a % b; a = b; b = t; }
    const int64_t step = groups / a, one = (units + 255) / 256;
    if (step > 4096) return 0;
    const int64_t want = one <= large ? one : large;
    const int64_t n = (want + step - 1) / step * step;
    return (uint32_t)(n > 4096 || (stream && n > large && 8 * (n - step) >= 7 * large) ? n - step : n);   // (4096: at most that many)
}

hawq_status launch_residual_add(int64_t n_pixels, int K, int m_dt, int r_dt, int y_dt, const void *m, const int32_t *m_b,
                                const uint8_t *m_c, const void *r, const int32_t *r_b, const uint8_t *r_c, int lo, int hi,
                                void *y, hipStream_t s) {
    const bool any4 = is4(m_dt) || is4(r_dt) || is4(y_dt);
    const uintptr_t al = (uintptr_t)m | (uintptr_t)r | (uintptr_t)y | (uintptr_t)m_b | (uintptr_t)r_b;
    if (!any4 && K % 4 == 0 && ((al & 15) | (((uintptr_t)m_c | (uintptr_t)r_c) & 3)) == 0 && n_pixels > 0) {
        const int64_t vu = n_pixels * (K / 4);
        // The streaming form from the size on at which its few, long-lived workgroups are no slower (operands not in L2, this form
        // against the other): with an INT32 operand 23 / 27 / 36 / 72 MB 6.5 / 7.3 / 7.8 / 13.5 us (7.0 / 7.6 / 9.0 / 16.2), but
        // 14 / 19 MB 5.3 / 5.6 (4.7 / 5.5); 8 bits both 4.8 / 9.6 / 19 MB 3.19 / 4.3 / 5.8 (3.26 / 4.75 / 7.1), 1.2 MB 2.70 (2.57).
        // INT32 operands past the caches from 128 MB in all on: between a layer that makes the INT32 operand and one that reads the sum,
        // 100 to 160 MB 4 % less of the three's time than with ordinary loads, above 160 2 to 13 %; below, the operands are still
        // in the caches (60 to 100 MB the addition by itself 1.15 times the ordinary loads' time, the three 1.00 to 1.05).
        auto bytes = [](int dt) { return dt == HAWQ_S32 ? 4 : 1; };
        const bool wide = m_dt == HAWQ_S32 || r_dt == HAWQ_S32, stream = vu >= (wide ? 900000 : 400000);
        const bool past = wide && vu * 4 * (bytes(m_dt) + bytes(r_dt) + bytes(y_dt)) >= 128000000;
        const uint32_t nb = grouped_blocks(vu, K / 4, stream ? 768 : 1024, stream);
        if (nb != 0) {
            auto go = [&](auto md, auto rd) {
                constexpr int MD = decltype(md)::value, RD = decltype(rd)::value;
                auto run = [&](auto kernel) { kernel<<<nb, 256, 0, s>>>((uint32_t)vu, K / 4, m, m_b, m_c, r, r_b, r_c, lo, hi, y); };
                if constexpr (MD == HAWQ_S32 || RD == HAWQ_S32)
                    if (stream && past) return y_dt == HAWQ_S32 ? run(residual_add_stream_kernel<MD, RD, true, true>) : run(residual_add_stream_kernel<MD, RD, false, true>);
                if (stream) y_dt == HAWQ_S32 ? run(residual_add_stream_kernel<MD, RD, true, false>) : run(residual_add_stream_kernel<MD, RD, false, false>);
                else y_dt == HAWQ_S32 ? run(residual_add_vec_kernel<MD, RD, true>) : run(residual_add_vec_kernel<MD, RD, false>);
            };
            auto on_r = [&](auto md) {
                if (r_dt == HAWQ_S32) go(md, std::integral_constant<int, HAWQ_S32>{});
                else if (r_dt == HAWQ_U8) go(md, std::integral_constant<int, HAWQ_U8>{});
                else go(md, std::integral_constant<int, HAWQ_S8>{});
            };
            if (m_dt == HAWQ_S32) on_r(std::integral_constant<int, HAWQ_S32>{});
            else if (m_dt == HAWQ_U8) on_r(std::integral_constant<int, HAWQ_U8>{});
            else on_r(std::integral_constant<int, HAWQ_S8>{});
            return check_launch();
        }
    }
    int per = (K % 4 == 0 && ((uintptr_t)y & 3) == 0) ? 4 : (any4 ? 2 : 1);
    const int64_t units = n_pixels * K / per;
    if (units == 0) return HAWQ_OK;
    const int64_t blocks = (units + 255) / 256;
    if (blocks > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
    residual_add_kernel<<<(uint32_t)blocks, 256, 0, s>>>(units, K, per, m_dt, r_dt, y_dt, m, m_b, m_c, r, r_b, r_c, lo, hi, y);
    return check_launch();
}

// ---- global average pool (Appendix E): INT32 sum over H*W, then one dyadic rescale ----
// grid: (ceil(C/per/64), N); one thread sums `per` adjacent channels over all pixels, so a
// wave reads 64*per consecutive bytes of every pixel.
__global__ void __launch_bounds__(64)
avgpool_kernel(const int HW, const int C, const int per, const int x_dt, const int y_dt, const void *__restrict__ x,
               const int32_t *__restrict__ b, const uint8_t *__restrict__ c, const int lo, const int hi, void *__restrict__ y) {
    const int n = blockIdx.y;
    const int k0 = (blockIdx.x * 64 + threadIdx.x) * per;
    if (k0 >= C) return;
    int32_t sum[4] = {0, 0, 0, 0};
    const int64_t base = (int64_t)n * HW * C + k0;
    if (per == 4 && !is4(x_dt)) {
        const uint8_t *xp = (const uint8_t *)x + base;
        for (int i = 0; i < HW; ++i) {
            const uint32_t v = *(const uint32_t *)(xp + (int64_t)i * C);
            if (x_dt == HAWQ_U8) {
                sum[0] += v & 0xff; sum[1] += (v >> 8) & 0xff; sum[2] += (v >> 16) & 0xff; sum[3] += v >> 24;
            } else {
                sum[0] += (int8_t)(v & 0xff); sum[1] += (int8_t)((v >> 8) & 0xff);
                sum[2] += (int8_t)((v >> 16) & 0xff); sum[3] += (int8_t)(v >> 24);
            }
        }
    } else {
        for (int i = 0; i < HW; ++i)
            for (int j = 0; j < per; ++j) sum[j] += load_elem(x, x_dt, base + (int64_t)i * C + j);
    }
    int32_t out[4];
    for (int j = 0; j < per; ++j) out[j] = clamp64(rq64(sum[j], b[k0 + j], c[k0 + j]), lo, hi);
    const int64_t o = (int64_t)n * C + k0;
    if (y_dt == HAWQ_S32) {
        for (int j = 0; j < per; ++j) ((int32_t *)y)[o + j] = out[j];
    } else if (is4(y_dt)) {
        for (int j = 0; j < per; j += 2) ((uint8_t *)y)[(o + j) >> 1] = (uint8_t)((out[j] & 0xf) | ((out[j + 1] & 0xf) << 4));
    } else {
        for (int j = 0; j < per; ++j) ((uint8_t *)y)[o + j] = (uint8_t)out[j];
    }
}

// fast path: unsigned 8-bit input, 8-bit output, C % 256 == 0.  A workgroup owns 256 channels of one image:
// 16 channel groups (16 bytes each) x 16 pixel slices; every thread adds up its slice's pixels with 16-byte
// loads, the 16 partial sums of a channel group meet in LDS, one thread per channel requantises.
__global__ void __launch_bounds__(256)
avgpool_u8_kernel(const int HW, const int C, const uint8_t *__restrict__ x, const int32_t *__restrict__ b,
                  const uint8_t *__restrict__ c, const int lo, const int hi, uint8_t *__restrict__ y) {
    __shared__ int32_t part[16][256 + 8];
    // (the XCDs take contiguous images, as the kernel that wrote them did)
    const uint32_t L = xcd_remap(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
    const int n = (int)(L / gridDim.x), cbase = (int)(L % gridDim.x) * 256;
    const int g = threadIdx.x & 15, sl = threadIdx.x >> 4;
    int32_t sum[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) sum[j] = 0;
    const uint8_t *xp = x + (int64_t)n * HW * C + cbase + g * 16;
    for (int i = sl; i < HW; i += 16) {
        const uint4 v = *(const uint4 *)(xp + (int64_t)i * C);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            sum[4 * d + 0] += w[d] & 0xff; sum[4 * d + 1] += (w[d] >> 8) & 0xff;
            sum[4 * d + 2] += (w[d] >> 16) & 0xff; sum[4 * d + 3] += w[d] >> 24;
        }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) part[sl][g * 16 + j] = sum[j];
    __syncthreads();
    const int k = threadIdx.x;   // one channel per thread
    int32_t t = 0;
#pragma unroll
    for (int s2 = 0; s2 < 16; ++s2) t += part[s2][k];
    y[(int64_t)n * C + cbase + k] = (uint8_t)clamp64(rq64(t, b[cbase + k], c[cbase + k]), lo, hi);
}

hawq_status launch_avgpool(int N, int HW, int C, int x_dt, int y_dt, const void *x, const int32_t *b, const uint8_t *c,
                           int lo, int hi, void *y, hipStream_t s) {
    if (N == 0) return HAWQ_OK;
    if (x_dt == HAWQ_U8 && (y_dt == HAWQ_U8 || y_dt == HAWQ_S8) && C % 256 == 0 && ((uintptr_t)x & 15) == 0) {
        dim3 grid(C / 256, N);
        avgpool_u8_kernel<<<grid, 256, 0, s>>>(HW, C, (const uint8_t *)x, b, c, lo, hi, (uint8_t *)y);
        return check_launch();
    }
    const bool any4 = is4(x_dt) || is4(y_dt);
    const int per = (C % 4 == 0 && ((uintptr_t)x & 3) == 0) ? 4 : (any4 ? 2 : 1);
    dim3 grid((C / per + 63) / 64, N);
    avgpool_kernel<<<grid, 64, 0, s>>>(HW, C, per, x_dt, y_dt, x, b, c, lo, hi, y);
    return check_launch();
}

// ---- max pool 3x3 / 2, pad 1 ----

// fast path: U8 in, C % 16 == 0; one thread = 16 channels of one output pixel
__global__ void __launch_bounds__(256)
maxpool_u8_kernel(const int64_t units, const int H, const int W, const int C, const int P, const int Q,
                  const uint8_t *__restrict__ x, const int lo, const int hi, const int y_dt, uint8_t *__restrict__ y) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= units) return;
    const int cg = C / 16;
    const int g = (int)(u % cg);
    int64_t t = u / cg;
    const int q = (int)(t % Q); t /= Q;
    const int p = (int)(t % P);
    const int n = (int)(t / P);
    uint4 best = make_uint4(0, 0, 0, 0);   // unsigned data: 0 is the identity, padding never wins
    for (int r = 0; r < 3; ++r) {
        const int ih = 2 * p - 1 + r;
        if (ih < 0 || ih >= H) continue;
        for (int s = 0; s < 3; ++s) {
            const int iw = 2 * q - 1 + s;
            if (iw < 0 || iw >= W) continue;
            const uint4 v = *(const uint4 *)(x + (((int64_t)n * H + ih) * W + iw) * C + g * 16);
            best.x = max_u8x4(best.x, v.x); best.y = max_u8x4(best.y, v.y);
            best.z = max_u8x4(best.z, v.z); best.w = max_u8x4(best.w, v.w);
        }
    }
    uint32_t wv[4] = {best.x, best.y, best.z, best.w};
    uint32_t ov[4];
    uint32_t nib[2] = {0, 0};
    for (int d = 0; d < 4; ++d) {
        uint32_t o = 0, h = 0;
        for (int j = 0; j < 4; ++j) {
            int32_t v = (int32_t)((wv[d] >> (8 * j)) & 0xff);
            v = v < lo ? lo : (v > hi ? hi : v);
            o |= (uint32_t)(v & 0xff) << (8 * j);
            h |= (uint32_t)(v & 0xf) << (4 * j);
        }
        ov[d] = o;
        nib[d >> 1] |= h << (16 * (d & 1));
    }
    const int64_t oe = (((int64_t)n * P + p) * Q + q) * C + g * 16;
    if (is4(y_dt)) *(uint2 *)(y + (oe >> 1)) = make_uint2(nib[0], nib[1]);
    else *(uint4 *)(y + oe) = make_uint4(ov[0], ov[1], ov[2], ov[3]);
}

__global__ void __launch_bounds__(256)
maxpool_generic_kernel(const int64_t units, const int per, const int H, const int W, const int C, const int P, const int Q,
                       const int x_dt, const int y_dt, const void *__restrict__ x, const int lo, const int hi,
                       void *__restrict__ y) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= units) return;
    const int cu = C / per;
    const int k0 = (int)(u % cu) * per;
    int64_t t = u / cu;
    const int q = (int)(t % Q); t /= Q;
    const int p = (int)(t % P);
    const int n = (int)(t / P);
    int32_t out[2];
    for (int j = 0; j < per; ++j) {
        int32_t best = INT32_MIN;
        for (int r = 0; r < 3; ++r) {
            const int ih = 2 * p - 1 + r;
            if (ih < 0 || ih >= H) continue;
            for (int s = 0; s < 3; ++s) {
                const int iw = 2 * q - 1 + s;
                if (iw < 0 || iw >= W) continue;
                const int32_t v = load_elem(x, x_dt, (((int64_t)n * H + ih) * W + iw) * C + k0 + j);
                best = v > best ? v : best;
            }
        }
        out[j] = best < lo ? lo : (best > hi ? hi : best);
    }
    const int64_t oe = (((int64_t)n * P + p) * Q + q) * C + k0;
    if (is4(y_dt)) ((uint8_t *)y)[oe >> 1] = (uint8_t)((out[0] & 0xf) | ((out[1] & 0xf) << 4));
    else
        for (int j = 0; j < per; ++j) ((uint8_t *)y)[oe + j] = (uint8_t)out[j];   // (per = 2 with a 4-bit input and an 8-bit output)
}

hawq_status launch_maxpool(int N, int H, int W, int C, int x_dt, int y_dt, const void *x, int lo, int hi, void *y,
                           hipStream_t s) {
    const int P = (H - 1) / 2 + 1, Q = (W - 1) / 2 + 1;
    if (N == 0) return HAWQ_OK;
    const bool fast = x_dt == HAWQ_U8 && (y_dt == HAWQ_U8 || y_dt == HAWQ_U4) && C % 16 == 0 &&
                      (((uintptr_t)x | (uintptr_t)y) & 15) == 0 && lo >= 0;
    if (fast) {
        const int64_t units = (int64_t)N * P * Q * (C / 16);
        const int64_t blocks = (units + 255) / 256;
        if (blocks > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
        maxpool_u8_kernel<<<(uint32_t)blocks, 256, 0, s>>>(units, H, W, C, P, Q, (const uint8_t *)x, lo, hi, y_dt, (uint8_t *)y);
    } else {
        const int per = (is4(x_dt) || is4(y_dt)) ? 2 : 1;
        const int64_t units = (int64_t)N * P * Q * (C / per);
        const int64_t blocks = (units + 255) / 256;
        if (blocks > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
        maxpool_generic_kernel<<<(uint32_t)blocks, 256, 0, s>>>(units, per, H, W, C, P, Q, x_dt, y_dt, x, lo, hi, y);
    }
    return check_launch();
}

// ---- window-sum pool carried in INT32 (Appendix E) ----
// one thread = `per` adjacent channels of one output pixel; the in-image taps are added in INT32 (64-bit while adding,
// the caller's contract keeps the sum inside INT32), then either stored raw or rescaled by one dyadic number and clamped
__global__ void __launch_bounds__(256)
pool_sum_kernel(const int64_t units, const int H, const int W, const int C, const int R, const int S, const int sh, const int sw,
                const int ph, const int pw, const int P, const int Q, const int per, const int x_dt, const int y_dt,
                const void *__restrict__ x, const int32_t *__restrict__ b, const uint8_t *__restrict__ c, const int lo, const int hi,
                void *__restrict__ y) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= units) return;
    const int cg = C / per;
    const int k0 = (int)(u % cg) * per;
    int64_t t = u / cg;
    const int q = (int)(t % Q); t /= Q;
    const int p = (int)(t % P);
    const int n = (int)(t / P);
    int64_t sum[4] = {0, 0, 0, 0};
    for (int r = 0; r < R; ++r) {
        const int ih = p * sh - ph + r;
        if (ih < 0 || ih >= H) continue;
        for (int s = 0; s < S; ++s) {
            const int iw = q * sw - pw + s;
            if (iw < 0 || iw >= W) continue;
            const int64_t e = (((int64_t)n * H + ih) * W + iw) * C + k0;
            if (per == 4 && x_dt == HAWQ_S32) {
                const v4i v = *(const v4i *)((const int32_t *)x + e);
                sum[0] += v[0]; sum[1] += v[1]; sum[2] += v[2]; sum[3] += v[3];
            } else if (per == 4 && x_dt == HAWQ_U8) {
                const uint32_t v = *(const uint32_t *)((const uint8_t *)x + e);
                sum[0] += v & 0xff; sum[1] += (v >> 8) & 0xff; sum[2] += (v >> 16) & 0xff; sum[3] += v >> 24;
            } else {
                for (int j = 0; j < per; ++j) sum[j] += load_elem(x, x_dt, e + j);
            }
        }
    }
    int32_t out[4];
    for (int j = 0; j < per; ++j)
        out[j] = b != nullptr ? clamp64(rq64((int32_t)sum[j], b[k0 + j], c[k0 + j]), lo, hi) : (int32_t)sum[j];
    const int64_t o = (((int64_t)n * P + p) * Q + q) * C + k0;
    if (y_dt == HAWQ_S32) {
        for (int j = 0; j < per; ++j) ((int32_t *)y)[o + j] = out[j];
    } else if (is4(y_dt)) {
        for (int j = 0; j < per; j += 2) ((uint8_t *)y)[(o + j) >> 1] = (uint8_t)((out[j] & 0xf) | ((out[j + 1] & 0xf) << 4));
    } else if (per == 4) {
        ((uint32_t *)y)[o >> 2] = (out[0] & 0xff) | ((out[1] & 0xff) << 8) | ((out[2] & 0xff) << 16) | ((uint32_t)out[3] << 24);
    } else {
        for (int j = 0; j < per; ++j) ((uint8_t *)y)[o + j] = (uint8_t)out[j];
    }
}

// fast path for the Inception pooling branch: 3x3 / stride 1 / pad 1 on INT32 (or unsigned 8-bit) data, C % 4 == 0.  One
// thread = 4 channels of a QT-wide, PT-high patch of output pixels.  It walks the PT + 2 input rows under the patch once:
// per row QT + 2 loads and the QT horizontal three-sums; an output row is the sum of the last three rows' horizontal sums
// (kept in a ring of three).  (PT + 2)(QT + 2) loads for PT QT outputs -- 2.25 per output at 4 x 4 instead of 9, which is
// what the vector-memory path, not HBM, limits in the general kernel.
template <bool X32, int QT, int PT>
__global__ void __launch_bounds__(256)
pool_sum3x3_kernel(const int64_t units, const int H, const int W, const int C, const int y_dt, const void *__restrict__ x,
                   const int32_t *__restrict__ b, const uint8_t *__restrict__ c, const int lo, const int hi, void *__restrict__ y) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= units) return;
    const int cg = C / 4, qb = (W + QT - 1) / QT, pb = (H + PT - 1) / PT;
    const int k0 = (int)(u % cg) * 4;
    int64_t t = u / cg;
    const int q0 = (int)(t % qb) * QT; t /= qb;
    const int p0 = (int)(t % pb) * PT;
    const int n = (int)(t / pb);
    int32_t bb[4] = {0, 0, 0, 0}, cc[4] = {1, 1, 1, 1};
    if (b != nullptr)
        for (int j = 0; j < 4; ++j) { bb[j] = b[k0 + j]; cc[j] = c[k0 + j]; }
    int32_t hs[3][QT][4];   // horizontal three-sums of the last three input rows
    static_for<0, PT + 2>([&](auto rc) {
        constexpr int rr = decltype(rc)::value;
        constexpr int slot = rr % 3;
        const int ih = p0 - 1 + rr;
        int32_t v[QT + 2][4];
#pragma unroll
        for (int j = 0; j < QT + 2; ++j) {
            const int iw = q0 - 1 + j;
            v[j][0] = v[j][1] = v[j][2] = v[j][3] = 0;
            if (ih < 0 || ih >= H || iw < 0 || iw >= W) continue;
            const int64_t e = (((int64_t)n * H + ih) * W + iw) * C + k0;
            if (X32) {
                const v4i w4 = *(const v4i *)((const int32_t *)x + e);
                v[j][0] = w4[0]; v[j][1] = w4[1]; v[j][2] = w4[2]; v[j][3] = w4[3];
            } else {
                const uint32_t w1 = *(const uint32_t *)((const uint8_t *)x + e);
                v[j][0] = w1 & 0xff; v[j][1] = (w1 >> 8) & 0xff; v[j][2] = (w1 >> 16) & 0xff; v[j][3] = w1 >> 24;
            }
        }
#pragma unroll
        for (int i = 0; i < QT; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) hs[slot][i][j] = v[i][j] + v[i + 1][j] + v[i + 2][j];
        if constexpr (rr >= 2) {
            const int p = p0 + rr - 2;
            if (p < H) {
#pragma unroll
                for (int i = 0; i < QT; ++i) {
                    if (q0 + i >= W) break;
                    int32_t out[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int32_t sum = hs[0][i][j] + hs[1][i][j] + hs[2][i][j];
                        out[j] = b != nullptr ? clamp64(rq64(sum, bb[j], cc[j]), lo, hi) : sum;
                    }
                    const int64_t o = (((int64_t)n * H + p) * W + q0 + i) * C + k0;
                    if (y_dt == HAWQ_S32) *(v4i *)((int32_t *)y + o) = (v4i){out[0], out[1], out[2], out[3]};
                    else if (is4(y_dt)) *(uint16_t *)((uint8_t *)y + (o >> 1)) = (uint16_t)((out[0] & 0xf) | ((out[1] & 0xf) << 4) | ((out[2] & 0xf) << 8) | ((out[3] & 0xf) << 12));
                    else ((uint32_t *)y)[o >> 2] = (out[0] & 0xff) | ((out[1] & 0xff) << 8) | ((out[2] & 0xff) << 16) | ((uint32_t)out[3] << 24);
                }
            }
        }
    });
}

hawq_status launch_pool_sum(int N, int H, int W, int C, int R, int S, int sh, int sw, int ph, int pw, int x_dt, int y_dt,
                            const void *x, const int32_t *b, const uint8_t *c, int lo, int hi, void *y, hipStream_t s) {
    const int P = (H + 2 * ph - R) / sh + 1, Q = (W + 2 * pw - S) / sw + 1;
    const bool any4 = is4(x_dt) || is4(y_dt);
    if (R == 3 && S == 3 && sh == 1 && sw == 1 && ph == 1 && pw == 1 && C % 4 == 0 && (x_dt == HAWQ_S32 || x_dt == HAWQ_U8) &&
        (((uintptr_t)x | (uintptr_t)y) & 15) == 0) {
        // patches of 4x4 outputs once they give every compute unit a workgroup (128 x 35 x 35 x 288 INT32: 4x4 73.8 us, 4x8 76.8,
        // 8x4 77.4, 8x8 78.2; one row of eight 117.6), smaller ones below (17 x 17 x 64 at batch 4: 7 workgroups of 4x4 patches
        // 7.4 us, 73 of single outputs 4.1).  INT32 maps of many channels, whose rows the smaller patches read more often from
        // beyond the L2s, from fewer workgroups on (35 x 35 x 768 at batch 4, 243 workgroups of 4x4: 10.0 us, 2x2 11.7; 28 x 28 x 1024,
        // 196: 9.6 and 11.2; at 183 9.5 and 8.8)
        auto blocks_of = [&](int t) { return ((int64_t)N * ((H + t - 1) / t) * ((W + t - 1) / t) * (C / 4) + 255) / 256; };
        if (N == 0) return HAWQ_OK;
        if (blocks_of(1) > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
        auto go = [&](auto tc) {
            constexpr int PT = decltype(tc)::value;
            const int64_t units = (int64_t)N * ((H + PT - 1) / PT) * ((W + PT - 1) / PT) * (C / 4);
            const uint32_t blocks = (uint32_t)blocks_of(PT);
            if (x_dt == HAWQ_S32) pool_sum3x3_kernel<true, PT, PT><<<blocks, 256, 0, s>>>(units, H, W, C, y_dt, x, b, c, lo, hi, y);
            else pool_sum3x3_kernel<false, PT, PT><<<blocks, 256, 0, s>>>(units, H, W, C, y_dt, x, b, c, lo, hi, y);
        };
        const int64_t large = x_dt != HAWQ_S32 || C < 512 ? 256 : C < 768 ? 240 : 192;
        if (blocks_of(4) >= large) go(std::integral_constant<int, 4>{});
        else if (blocks_of(2) >= 256) go(std::integral_constant<int, 2>{});
        else go(std::integral_constant<int, 1>{});
        return check_launch();
    }
    const int per = (C % 4 == 0 && (((uintptr_t)x | (uintptr_t)y) & 15) == 0) ? 4 : (any4 ? 2 : 1);
    const int64_t units = (int64_t)N * P * Q * (C / per);
    if (units == 0) return HAWQ_OK;
    const int64_t blocks = (units + 255) / 256;
    if (blocks > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
    pool_sum_kernel<<<(uint32_t)blocks, 256, 0, s>>>(units, H, W, C, R, S, sh, sw, ph, pw, P, Q, per, x_dt, y_dt, x, b, c, lo, hi, y);
    return check_launch();
}

// ---- concatenation with one dyadic number per branch (Appendix E) ----
// one launch per branch: branch elements [n_pixels][K] -> channels off .. off + K of the [n_pixels][Kt] output
__global__ void __launch_bounds__(256)
concat_branch_kernel(const int64_t units, const int K, const int Kt, const int off, const int per, const int q_dt, const int y_dt,
                     const void *__restrict__ q, const int32_t *__restrict__ b, const uint8_t *__restrict__ c, const int lo, const int hi,
                     void *__restrict__ y) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u >= units) return;
    const int kg = K / per;
    const int64_t px = u / kg;
    const int k0 = (int)(u - px * kg) * per;
    const int64_t e = px * K + k0;
    int32_t out[4];
    if (per == 4 && q_dt == HAWQ_S32) {
        const v4i v = *(const v4i *)((const int32_t *)q + e);
        for (int j = 0; j < 4; ++j) out[j] = clamp64(rq64(v[j], b[k0 + j], c[k0 + j]), lo, hi);
    } else {
        for (int j = 0; j < per; ++j) out[j] = clamp64(rq64(load_elem(q, q_dt, e + j), b[k0 + j], c[k0 + j]), lo, hi);
    }
    const int64_t o = px * Kt + off + k0;
    if (y_dt == HAWQ_S32) {
        for (int j = 0; j < per; ++j) ((int32_t *)y)[o + j] = out[j];
    } else if (is4(y_dt)) {
        for (int j = 0; j < per; j += 2) ((uint8_t *)y)[(o + j) >> 1] = (uint8_t)((out[j] & 0xf) | ((out[j + 1] & 0xf) << 4));
    } else if (per == 4) {
        ((uint32_t *)y)[o >> 2] = (out[0] & 0xff) | ((out[1] & 0xff) << 8) | ((out[2] & 0xff) << 16) | ((uint32_t)out[3] << 24);
    } else {
        for (int j = 0; j < per; ++j) ((uint8_t *)y)[o + j] = (uint8_t)out[j];
    }
}

// Vector form, all branches in one launch: every K_i and offset a multiple of four, INT32 or 8-bit branches and outputs
// (also packed 4-bit outputs).  A thread keeps one group of four output channels -- its branch and parameters are looked up
// once -- and walks pixels with four loads in flight.  Bound: HBM (every branch and the output once).
constexpr int kConcatMax = 8;
struct ConcatArgs {
    const void *q[kConcatMax];
    const int32_t *b[kConcatMax];
    const uint8_t *c[kConcatMax];
    uint32_t end[kConcatMax];      // first channel group past the branch
    int32_t dt[kConcatMax];
};
// MANY: the form of large tensors, which eight waves a SIMD walk: its 64-bit evaluation has two pixels in flight, not four, and
// the kernel 64 registers instead of 94 (with five waves a SIMD see launch_concat_all; with c > 32 in every channel it is 2 to
// 12 % slower than four pixels in flight at eight waves were, 60 to 130 MB).
template <int YB, bool MANY>   // bits of an output element
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MANY ? 8 : 5)))
concat_vec_kernel(const ConcatArgs a, const int n, const uint32_t units, const uint32_t groups, const int lo, const int hi, void *y) {
    constexpr int U = 4;
    const uint32_t T = gridDim.x * 256;
    uint32_t u = blockIdx.x * 256 + threadIdx.x;
    const uint32_t px0 = u / groups, g = u - px0 * groups, dpx = T / groups;
    int i = 0;
    uint32_t begin = 0;
#pragma unroll
    for (int j = 0; j < kConcatMax - 1; ++j)
        if (j < n - 1 && g >= a.end[j]) { i = j + 1; begin = a.end[j]; }
    const void *q = a.q[0];
    const int32_t *bp = a.b[0];
    const uint8_t *cp = a.c[0];
    int dt = a.dt[0];
    uint32_t end = a.end[0];
#pragma unroll
    for (int j = 1; j < kConcatMax; ++j)
        if (i == j) { q = a.q[j]; bp = a.b[j]; cp = a.c[j]; dt = a.dt[j]; end = a.end[j]; }
    const uint32_t w = end - begin, k = g - begin;
    auto load = [&](uint32_t at) { return dt == HAWQ_S32 ? load4<HAWQ_S32>(q, at) : dt == HAWQ_U8 ? load4<HAWQ_U8>(q, at) : load4<HAWQ_S8>(q, at); };
    const v4i b = ((const v4i *)bp)[k];
    const uint32_t c = ((const uint32_t *)cp)[k];
    uint32_t e = px0 * w + k;
    const uint32_t de = dpx * w;
    v4i v[U];
    auto fetch = [&]() -> bool {       // four pixels' values, or the one that is left
        const bool four = u + (U - 1) * T < units;
        if (u < units) v[0] = load(e);
        if (four)
#pragma unroll
            for (int j = 1; j < U; ++j) v[j] = load(e + j * de);
        return four;
    };
    bool four = fetch();               // (in flight while the parameters arrive and their form is decided)
    // narrow evaluation in its INT32 form for either operand width (see Rescale4)
    Rescale4<HAWQ_S32> pq;
    const bool narrow = pq.init(b, c);
    int32_t vlo = lo, vhi = hi;
    int64_t half = (int64_t)1 << 31;
    asm volatile("" : "+v"(vlo), "+v"(vhi), "+v"(half));
    auto put = [&](const v4i &o, uint32_t at) {
        if constexpr (YB == 32) ((v4i *)y)[at] = o;
        else if constexpr (YB == 8) ((uint32_t *)y)[at] = pack4(o);
        else ((uint16_t *)y)[at] = (uint16_t)((o[0] & 0xf) | ((o[1] & 0xf) << 4) | ((o[2] & 0xf) << 8) | ((o[3] & 0xf) << 12));
    };
    auto walk = [&](auto nc) {
        auto finish = [&](const v4i &v, uint32_t at) {
            v4i o;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (decltype(nc)::value) o[j] = med3(pq.narrow(v[j], j, half), vlo, vhi);
                else o[j] = clamp64(pq.wide(v[j], j), lo, hi);
            }
            put(o, at);
        };
        while (four) {
#pragma unroll
            for (int j = 0; j < U; ++j) finish(v[j], u + j * T);
            u += U * T;
            e += U * de;
            four = fetch();
        }
        while (u < units) {
            finish(v[0], u);
            u += T;
            e += de;
            if (u < units) v[0] = load(e);
        }
    };
    if (__all(narrow)) walk(std::true_type{});
    else if constexpr (!MANY) walk(std::false_type{});
    else {
        auto unit = [&](const v4i &t, uint32_t at) {
            v4i o;
            uint32_t cs = c;
            asm volatile("" : "+v"(cs));       // (kept over the loop, the shifts' 64-bit roundings alone are sixteen registers)
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = clamp64(rq64(t[j], b[j], (cs >> (8 * j)) & 0xff), lo, hi);
            put(o, at);
        };
#pragma unroll 1
        for (; u + T < units; u += 2 * T, e += 2 * de) {
            const v4i t0 = load(e), t1 = load(e + de);
            unit(t0, u);
            unit(t1, u + T);
        }
        if (u < units) unit(load(e), u);
    }
}

bool launch_concat_all(int64_t n_pixels, int n, const hawq_concat_branch *br, int Kt, int y_dt, int lo, int hi, void *y, hipStream_t s,
                       hawq_status &st) {
    if (n > kConcatMax || Kt % 4 != 0 || ((uintptr_t)y & 15) != 0 || n_pixels == 0) return false;
    // One INT32 branch to 8 or 4 bits -- a tensor requantised -- has no branch to look up and no second launch to save: the
    // form of one group of channels per thread is the faster for short tensors (P x K = 4900 x 64 2.9 us, 3.15 here; from 2^19
    // groups on 4900 x 1024 6.0 and 5.6, packed 6.6 and 5.3) and, to 8 bits, for very long ones (39200 x 2048 76 us, 85 here).
    const int64_t groups_all = n_pixels * (Kt / 4);
    if (n == 1 && br[0].dtype == HAWQ_S32 && y_dt != HAWQ_S32 && (groups_all < (1 << 19) || (!is4(y_dt) && groups_all > (1 << 24)))) return false;
    ConcatArgs a{};
    uint32_t end = 0;
    for (int i = 0; i < n; ++i) {
        if (br[i].K % 4 != 0 || is4(br[i].dtype) || (((uintptr_t)br[i].q | (uintptr_t)br[i].b) & 15) || ((uintptr_t)br[i].c & 3)) return false;
        end += br[i].K / 4;
        a.q[i] = br[i].q; a.b[i] = br[i].b; a.c[i] = br[i].c; a.end[i] = end; a.dt[i] = br[i].dtype;
    }
    // From 2^22 groups on (some 60 MB) 4096 workgroups of the form with eight waves a SIMD: the others' five have too few bytes in
    // flight there, of 8-bit branches above all.  285 shapes against the 64-bit form with a workgroup to each four units: 60 to 80 MB
    // 0.97 -> 0.91 of its time, 80 to 160 1.02 to 1.05 -> 0.91, above 1.07 -> 0.95 (single shapes 1.21 -> 1.00).  Below, the fewer
    // workgroups are as fast or faster (20 to 40 MB 0.84 of that time, with 4096 0.88).
    const int64_t units = n_pixels * (Kt / 4);
    const bool many = units >= 1 << 22;
    const uint32_t nb = grouped_blocks(units, Kt / 4, many ? 4096 : 1024);
    if (nb == 0) return false;
    auto run = [&](auto kernel) { kernel<<<nb, 256, 0, s>>>(a, n, (uint32_t)units, Kt / 4, lo, hi, y); };
    if (y_dt == HAWQ_S32) many ? run(concat_vec_kernel<32, true>) : run(concat_vec_kernel<32, false>);
    else if (is4(y_dt)) many ? run(concat_vec_kernel<4, true>) : run(concat_vec_kernel<4, false>);
    else many ? run(concat_vec_kernel<8, true>) : run(concat_vec_kernel<8, false>);
    st = check_launch();
    return true;
}

hawq_status launch_concat_branch(int64_t n_pixels, int K, int Kt, int off, int q_dt, int y_dt, const void *q, const int32_t *b,
                                 const uint8_t *c, int lo, int hi, void *y, hipStream_t s) {
    const bool any4 = is4(q_dt) || is4(y_dt);
    // four channels per thread need dword-aligned output positions (and 16-byte aligned INT32 rows)
    const bool vec = K % 4 == 0 && Kt % 4 == 0 && off % 4 == 0 && (((uintptr_t)q | (uintptr_t)y) & 15) == 0;
    const int per = vec ? 4 : (any4 ? 2 : 1);
    const int64_t units = n_pixels * (K / per);
    if (units == 0) return HAWQ_OK;
    const int64_t blocks = (units + 255) / 256;
    if (blocks > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
    concat_branch_kernel<<<(uint32_t)blocks, 256, 0, s>>>(units, K, Kt, off, per, q_dt, y_dt, q, b, c, lo, hi, y);
    return check_launch();
}

// ---- weights into the blocked order of the implicit-GEMM kernel: one thread per 16-byte chunk of the copy ----
__global__ void __launch_bounds__(256)
block_weights_kernel(const uint8_t *__restrict__ w, uint8_t *__restrict__ out, const int K, const int64_t row, const int64_t chunks) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= chunks) return;
    const int64_t steps = row / 64;
    const int ch = (int)(i & 3);
    const int kk = (int)((i >> 2) & 63);
    const int64_t blk = i >> 8;                  // (k / 64) * steps + step
    const int64_t st = blk % steps;
    const int k = (int)(blk / steps) * 64 + kk;
    v4i v = {0, 0, 0, 0};
    if (k < K) v = *(const v4i *)(w + (int64_t)k * row + st * 64 + ch * 16);
    *(v4i *)(out + i * 16) = v;
}

hawq_status launch_block_weights(const void *w, void *w_blocked, int K, int64_t row, hipStream_t s) {
    const int64_t chunks = (int64_t)((K + 63) / 64) * (row / 64) * 256;
    if (chunks == 0) return HAWQ_OK;
    const int64_t blocks = (chunks + 255) / 256;
    if (blocks > 0x7fffffff) return HAWQ_ERR_UNSUPPORTED;
    block_weights_kernel<<<(uint32_t)blocks, 256, 0, s>>>((const uint8_t *)w, (uint8_t *)w_blocked, K, row, chunks);
    return check_launch();
}

}  // namespace hawq
