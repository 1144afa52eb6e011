// dense_step.h -- one 32-token step of attention over 16-bit rows on the
// gfx950 matrix cores, shared by the dense kernel and by the decode kernel's
// blocks that keep every channel (not part of the C ABI).
#pragma once
#include "mosaic_internal.h"

namespace mosaic {

constexpr int DSTEP = 32;                 // tokens of a wave's step

typedef __attribute__((ext_vector_type(8))) __bf16 dbf8;
typedef __attribute__((ext_vector_type(8))) _Float16 dhf8;
typedef __attribute__((ext_vector_type(4))) float df4;
typedef __attribute__((ext_vector_type(4))) uint32_t du4;

template <int DT> struct DMma;
template <> struct DMma<1> {
    using v8 = dbf8;
    using el = __bf16;
    static __device__ __forceinline__ df4 run(v8 a, v8 b, df4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
template <> struct DMma<0> {
    using v8 = dhf8;
    using el = _Float16;
    static __device__ __forceinline__ df4 run(v8 a, v8 b, df4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};

// maximum / sum over the four lanes l, l ^ 16, l ^ 32, l ^ 48
template <typename F>
__device__ __forceinline__ float rows_all(float x, F f) {
    uint32_t u = __float_as_uint(x);
    const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    x = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
    u = __float_as_uint(x);
    const auto b = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Four channel tiles of the second product's right operand: each lane's two
// transposing reads of a tile are 4 tokens of one channel, 16 rows (4096
// bytes) apart.  Written out, with their wait: the compiler, which does not
// tell the buffer being filled from the one being read, would wait for the
// next step's direct loads before every one.
template <typename M8>
__device__ __forceinline__ void read_tr4(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, M8 (&b)[4]) {
    uint64_t w[8];
    asm volatile("ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:4096\n\t"
                 "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:4096\n\t"
                 "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:4096\n\t"
                 "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:4096\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
                 : "v"(a0), "v"(a1), "v"(a2), "v"(a3)
                 : "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i) __builtin_memcpy(&b[i], &w[2 * i], 16);
}

// LDS addresses of the transposing reads of each channel tile, for V rows of
// 256 bytes at base whose 16-byte piece c sits at piece c ^ (row % 16)
__device__ __forceinline__ void tr_addresses(uint32_t base, uint32_t (&va)[8]) {
    const int lane = threadIdx.x & 63, l16 = lane & 15, r = 4 * (lane >> 4) + (l16 >> 2);
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
        const int c = 2 * ct + ((l16 & 3) >> 1);
        va[ct] = base + (uint32_t)(r * 256 + 16 * (c ^ r) + 8 * (l16 & 1));
    }
}

// The online softmax of a step's logits z (token 16 n + 4 q4 + r, head l16)
// and its weights' product with the step's V rows, added to acc ([channel
// tile][row 4 q4 + r]).  The weights are the rows of the product's left
// operand in NPART 16-bit parts: rows h < GP the leading part, rows GP + h the
// residual, with three parts also the residual's residual (rows 2 GP + h, or a
// second product where GP is 8); ps scales them (1, or a power of two that
// keeps small weights in fp16's normal range).  ready() waits for the rows.
template <int DT, int GP, int NPART, typename R>
__device__ __forceinline__ void dense_accumulate(float (&z)[2][4], float &m_run, float &l_run, df4 (&acc)[8], float ps,
                                                 R ready, const uint32_t (&va)[8], uint32_t off) {
    using M8 = typename DMma<DT>::v8;
    using E = typename DMma<DT>::el;
    const int lane = threadIdx.x & 63, l16 = lane & 15, q4 = lane >> 4;
    float cm = -INFINITY;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) cm = fmaxf(cm, z[n][r]);
    cm = rows_all(cm, [](float a, float b) { return fmaxf(a, b); });
    const float mn = fmaxf(m_run, cm);
    const float mb = mn == -INFINITY ? 0.0f : mn;          // no token but masked ones (logit -inf) yet: weights 0
    const float alpha = __expf(m_run - mb);
    float ls = 0.0f;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z[n][r] = __expf(z[n][r] - mb);
            ls += z[n][r];
        }
    ls = rows_all(ls, [](float a, float b) { return a + b; });
    l_run = l_run * alpha + ls;
    m_run = mn;
    if (!__all(alpha == 1.0f)) {                           // some head's running maximum moved
        float ar[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {                      // alpha of head (4 q4 + r) % GP
            const float a0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha), r));
            if (GP == 4) ar[r] = a0;
            else {
                const float a1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha), 4 + r));
                ar[r] = (q4 & 1) ? a1 : a0;
            }
        }
#pragma unroll
        for (int ct = 0; ct < 8; ++ct)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[ct][r] *= ar[r];
    }
    M8 pa, pb{};                                           // inner index (q4, i): token 16 (i / 4) + 4 q4 + i % 4
    {
        M8 hi, mid, lo{};
        float rest[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) { const float x = z[i >> 2][i & 3] * ps; hi[i] = (E)x; rest[i] = x - (float)hi[i]; }
#pragma unroll
        for (int i = 0; i < 8; ++i) { mid[i] = (E)rest[i]; rest[i] = rest[i] - (float)mid[i]; }
        if (NPART == 3)
#pragma unroll
            for (int i = 0; i < 8; ++i) lo[i] = (E)rest[i];
        du4 wh = __builtin_bit_cast(du4, hi), wm = __builtin_bit_cast(du4, mid), wl = __builtin_bit_cast(du4, lo);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t m = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wm[e], 0x110 + GP, 0xf, 0xf, false);
            uint32_t w = l16 < GP ? wh[e] : m;
            if (NPART == 3 && GP == 4) {
                const uint32_t x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)wl[e], 0x118, 0xf, 0xf, false);
                w = l16 < 8 ? w : x;
            }
            wh[e] = w;
            if (GP == 8) wl[e] = l16 < GP ? wl[e] : 0u;
        }
        pa = __builtin_bit_cast(M8, wh);
        pb = __builtin_bit_cast(M8, wl);
    }
    ready();
#pragma unroll
    for (int c4 = 0; c4 < 8; c4 += 4) {
        M8 b[4];
        read_tr4(va[c4] + off, va[c4 + 1] + off, va[c4 + 2] + off, va[c4 + 3] + off, b);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            acc[c4 + c] = DMma<DT>::run(pa, b[c], acc[c4 + c]);
            if (NPART == 3 && GP == 8) acc[c4 + c] = DMma<DT>::run(pb, b[c], acc[c4 + c]);
        }
    }
}

}  // namespace mosaic
