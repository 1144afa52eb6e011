// encode.hip -- gfx950 kernel of the prefill's encoding pass for the kept
// counts 16, 32 and 48 (Sec. 4.2 stage 1, Sec. 4.3, Sec. 5.1, Sec. 5.2,
// Sec. 5.5): rotation, strategy search, packing and block keys of one
// 64-token segment per workgroup, wave 0 its keys and wave 1 its values.
//
// A lane holds one token's 128 rotated channels in registers, so a rank, a
// dropped energy or a bitmap of 64 vectors costs one instruction per step and
// no cross-lane traffic:
//   - rotation on the matrix cores in fp32.  v_mfma_f32_32x32x2_f32 adds its
//     two products as two fused multiply-adds in ascending k, one rounding
//     each, so a chain of 64 of them is bit for bit the fp32 fused chain over
//     ascending channels;
//   - the r largest group scores by sorting networks on registers (one
//     v_max / v_min pair per comparator): they give the r-th and (r + 1)-th
//     largest score of every candidate, and a group is kept when its score
//     reaches the r-th; where the two are equal a pass in channel order
//     breaks the tie by the lower index;
//   - the candidates are taken in order, each group size's network when it is
//     first needed, and stop at the first that passes for K and V.
// What bounds it: vector-ALU time.  The rotation's 512 matrix instructions take
// 33 K cycles of a wave (fp32 products run at twice the rate of plain fp32
// FMAs, but a wave's products and another wave's vector instructions were
// measured not to overlap: 225 + 262 us apart, 487 us together), the ranking
// and packing 14 K (first candidate passes) to 38 K, and the two make up 98 %
// of the time.  Two waves per SIMD (256 registers) hide the loads and barriers;
// spilled registers cost far more than their instructions say (110 of them 40 %
// of the forced strategy's time), hence the ordering constraints below.
// 2 x 131072 tokens, 8 kv heads, bf16: ranks counted through LDS, lane per
// channel, took 16.8 ms; this kernel takes 2.09 ms.  4 x 32785 tokens in fp16,
// first candidate: 6.87 ms and 0.88 ms.
#include <utility>

#include "mosaic_internal.h"

namespace mosaic {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int YH = D / 2;                 // channels staged at a time for the block means
constexpr int YB_STRIDE = YH + 2;         // floats per staged token row (8-byte aligned, banks 2 apart)
constexpr int MEAN_STRIDE = D + 4;        // floats per mean row (16-byte reads of 16 rows spread over the banks)
constexpr int MEAN_ROWS = 4 + 8 + 16;     // blocks of 16, then of 8, then of 4
constexpr int ST_MAX = 2 * 48 + 4;        // staged bytes of a token's kept values, at most

struct EncSmem {
    // keys: half of the rotated channels of every token, then the staged records
    float yb[SEG * YB_STRIDE];
    float mean[MEAN_ROWS * MEAN_STRIDE];
    uint8_t vst[SEG * ST_MAX];            // the staged records of the values
    uint32_t pass[12][2];                 // per exchange: candidates that pass for K, for V
    int log2b;
};
static_assert(sizeof(float) * SEG * YB_STRIDE >= SEG * ST_MAX, "the keys' staged records fit their channels' place");
static_assert(sizeof(float) * SEG * YB_STRIDE >= SEG * D * 2 &&
              sizeof(float) * MEAN_ROWS * MEAN_STRIDE + SEG * ST_MAX >= SEG * D * 2, "each wave's input rows");
static_assert(sizeof(EncSmem) * 4 <= 160 * 1024, "four workgroups per compute unit");

__device__ __forceinline__ int enc_log2(int v) { return 31 - __clz(v); }
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
}

// first row of the means of blocks of 2^log2b tokens
__device__ __forceinline__ int mean_row0(int log2b) { return log2b == 4 ? 0 : (log2b == 3 ? 4 : 12); }

// ------------------------------------------------------------------ rotation
// y[c] = rotated channel c of token `lane` of the segment at src.  Rows of
// the matrix product are the output channels, columns the tokens (32 per
// product, two products).  Row i of product rb is channel 4 i + rb, so a
// lane's four operands of a step are one 16-byte read of R^T; a lane then
// holds 64 channels of two tokens, and one swap of the wave's halves per
// register leaves all 128 channels of its own token.
//
// xs (16 KB of LDS, the wave's own) receives the input rows by direct loads,
// 16-byte piece k of row t at piece k ^ (t % 16) so that the lanes' reads of
// one piece spread over the banks; R^T streams through RING registers.  Both
// start before the first product: loads complete in order, so a wait on R^T
// behind loads of x from HBM would wait for those too (one 16-byte piece of x
// per lane and step in registers, 2 steps of R^T ahead: the products then
// took 110 K cycles of a wave's 144 K).
template <int DT>
__device__ __forceinline__ void rotate_rows(const uint16_t *src, const float *rt, uint8_t *xs, float (&y)[D]) {
    const int lane = threadIdx.x & 63, l32 = lane & 31, hl = lane >> 5;
    typedef __attribute__((address_space(3))) uint8_t lds_b;
    typedef __attribute__((address_space(1))) const uint8_t gl_b;
#pragma unroll
    for (int k = 0; k < 16; ++k) {                          // rows 4 k .. 4 k + 3
        const int t = 4 * k + (lane >> 4);
        __builtin_amdgcn_global_load_lds((gl_b *)(src + (uint64_t)t * D + 8 * ((lane & 15) ^ (t & 15))),
                                         (lds_b *)(xs + 1024 * k), 16, 0, 0);
    }
    constexpr int RING = 8;
    const float4 *ap = (const float4 *)rt + hl * (D / 4) + l32;       // + 2 (D / 4) per step
    float4 ar[RING];
#pragma unroll
    for (int i = 0; i < RING; ++i) ar[i] = ap[i * (2 * (D / 4))];
    f32x16 acc[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int rb = 0; rb < 4; ++rb) acc[t][rb] = f32x16{};
    const uint32_t sel = hl ? 0x03020c0cu : 0x01000c0cu;
    // channel 2 s + hl of a token, from the dword holding channels 2 s and 2 s + 1
    auto elem = [&](uint32_t w) -> float {
        if (DT) return __uint_as_float(__builtin_amdgcn_perm(0u, w, sel));
        return (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> (16 * hl)));
    };
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // piece k (8 channels, 4 steps) of tokens l32 and l32 + 32 (the same piece position: 32 % 16 = 0)
    const uint8_t *xr = xs + l32 * 256;
    auto piece = [&](int k) { return 16 * (k ^ (l32 & 15)); };
    uint4 xa = *(const uint4 *)(xr + piece(0)), xb = *(const uint4 *)(xr + 8192 + piece(0));
#pragma unroll 1
    for (int cb = 0; cb < 8; ++cb) {                         // 16 channels: two pieces, eight steps
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kn = piece(min(2 * cb + h + 1, 15));
            const uint4 na = *(const uint4 *)(xr + kn), nb = *(const uint4 *)(xr + 8192 + kn);
            const uint32_t wa[4] = {xa.x, xa.y, xa.z, xa.w}, wb[4] = {xb.x, xb.y, xb.z, xb.w};
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int i = 4 * h + s;
                const float4 a = ar[i];
                const float b0 = elem(wa[s]), b1 = elem(wb[s]);
                acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b0, acc[0][0], 0, 0, 0);
                acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b1, acc[1][0], 0, 0, 0);
                acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b0, acc[0][1], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b1, acc[1][1], 0, 0, 0);
                acc[0][2] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b0, acc[0][2], 0, 0, 0);
                acc[1][2] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b1, acc[1][2], 0, 0, 0);
                acc[0][3] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b0, acc[0][3], 0, 0, 0);
                acc[1][3] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b1, acc[1][3], 0, 0, 0);
                ar[i] = ap[min(RING * (cb + 1) + i, 63) * (2 * (D / 4))];
                __builtin_amdgcn_sched_barrier(0);
            }
            xa = na; xb = nb;
        }
    }
    // element v of product rb is row 8 (v / 4) + 4 (lane / 32) + v % 4
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[0][rb][v]), __float_as_uint(acc[1][rb][v]),
                                                            false, false);
            const int c = 32 * (v >> 2) + 4 * (v & 3) + rb;
            y[c] = __uint_as_float(r[0]);
            y[c + 16] = __uint_as_float(r[1]);
        }
}

// the unrotated row of token `lane`
template <int DT>
__device__ __forceinline__ void plain_rows(const uint16_t *src, float (&y)[D]) {
    const uint4 *x = (const uint4 *)(src + (uint64_t)(threadIdx.x & 63) * D);
#pragma unroll
    for (int k = 0; k < D / 8; ++k) {
        const uint4 t = x[k];
        const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) y[8 * k + e] = h2f((uint16_t)((e & 1) ? (w[e >> 1] >> 16) : w[e >> 1]), DT);
    }
}

// The channels as values the compiler knows nothing about: what one phase
// derives from them (squares, scores) is derived again in the next instead of
// being kept in registers that are not there.
__device__ __forceinline__ void renew(float (&y)[D]) {
#pragma unroll
    for (int i = 0; i < D; ++i) asm volatile("" : "+v"(y[i]));
}

// one channel, the same way (for the rare side of a branch, so that nothing of
// it is computed ahead of the branch)
__device__ __forceinline__ float aside(float x) {
    float o;
    asm volatile("" : "=v"(o) : "0"(x));
    return o;
}
// the channels of a group, read through aside() when ASIDE is set
template <bool ASIDE>
__device__ __forceinline__ float chan(const float (&y)[D], int i) { return ASIDE ? aside(y[i]) : y[i]; }

// every N steps: the scheduler moves nothing across (bounds what it computes ahead)
template <int I, int N>
__device__ __forceinline__ void bound_ahead() {
    if constexpr (I % N == 0) __builtin_amdgcn_sched_barrier(0);
}

// pairwise adjacent tree of N leaves from leaf B on, leaves taken in ascending order
template <int B, int N, typename F>
__device__ __forceinline__ float leaf_tree(F &f) {
    if constexpr (N == 1) return f(std::integral_constant<int, B>{});
    else {
        const float a = leaf_tree<B, N / 2>(f);
        const float b = leaf_tree<B + N / 2, N / 2>(f);
        return a + b;
    }
}

// ------------------------------------------------------------------ sorting networks (descending)
__device__ __forceinline__ void cas(int &a, int &b) {
    const int hi = max(a, b), lo = min(a, b);
    a = hi; b = lo;
}
// Batcher's odd-even merge of a[LO..HI] (step R); positions at or past LIM
// hold nothing (below everything), so their comparators do nothing
template <int LO, int HI, int R, int LIM, int N>
__device__ __forceinline__ void oe_merge(int (&a)[N]) {
    if constexpr (2 * R < HI - LO) {
        oe_merge<LO, HI, 2 * R, LIM>(a);
        oe_merge<LO + R, HI, 2 * R, LIM>(a);
#pragma unroll
        for (int i = LO + R; i < HI - R; i += 2 * R)
            if (i + R < LIM) cas(a[i], a[i + R]);
    } else if constexpr (LO + R < LIM) {
        cas(a[LO], a[LO + R]);
    }
}
template <int LO, int HI, int N>
__device__ __forceinline__ void oe_sort(int (&a)[N]) {
    if constexpr (HI > LO) {
        constexpr int M = (LO + HI) / 2;
        oe_sort<LO, M>(a);
        oe_sort<M + 1, HI>(a);
        oe_merge<LO, HI, 1, N>(a);
    }
}
// a bitonic run a[LO .. LO + N) into descending order
template <int LO, int N, int M>
__device__ __forceinline__ void bitonic_desc(int (&a)[M]) {
    if constexpr (N > 1) {
#pragma unroll
        for (int i = 0; i < N / 2; ++i) cas(a[LO + i], a[LO + N / 2 + i]);
        bitonic_desc<LO, N / 2>(a);
        bitonic_desc<LO + N / 2, N / 2>(a);
    }
}

// Scores as integers (the bits of a non-negative float order like the
// float), -1 for the groups past the truncation.
struct Trunc {
    int m[4];                             // per 32 channels: 0, or -1 past the truncation
};
template <int G, int I, bool ASIDE = false>
__device__ __forceinline__ int group_key(const float (&y)[D], const Trunc &tr) {
    auto a = [&](int i) { return fabsf(chan<ASIDE>(y, G * I + i)); };
    float s;
    if constexpr (G == 1) s = a(0);
    else if constexpr (G == 2) s = a(0) + a(1);
    else s = (a(0) + a(1)) + (a(2) + a(3));
    if constexpr (G == 1 && !ASIDE) {                       // magnitude and truncation in one operation
        int k;
        asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(k) : "v"(y[I]), "s"(0x7fffffff), "v"(tr.m[I / 32]));
        return k;
    }
    return __float_as_int(s) | tr.m[G * I / 32];
}
template <int G, int A, int N, int M, int... I>
__device__ __forceinline__ void load_keys(const float (&y)[D], const Trunc &tr, int (&k)[M], int at, std::integer_sequence<int, I...>) {
    ((k[at + I] = group_key<G, A + I>(y, tr)), ...);
}
template <int G, int A, int N, int M>
__device__ __forceinline__ void load_keys(const float (&y)[D], const Trunc &tr, int (&k)[M], int at) {
    load_keys<G, A, N>(y, tr, k, at, std::make_integer_sequence<int, N>{});
}

// per candidate kept count (16, 32, 48): the score of the last group kept and
// the largest score left out
struct Cuts {
    int t[3], nx[3];
};

// The cuts of 16 and 32 kept single channels: the 32 largest so far stay
// sorted and the last 32 only meet the list, since the 16th and 17th of a
// bitonic 32 are a half-cleaner away (2150 vector instructions; with the 48
// largest below, 2800).
__device__ __forceinline__ Cuts cuts32(const float (&y)[D], const Trunc &tr) {
    Cuts c;
    int l[32], rest = -1;
    load_keys<1, 0, 32>(y, tr, l, 0);
    oe_sort<0, 31>(l);
    auto meet = [&](auto first) {                            // l: the 32 largest of it and 32 more, bitonic
        int n[32];
        load_keys<1, decltype(first)::value, 32>(y, tr, n, 0);
        oe_sort<0, 31>(n);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            rest = max(rest, min(l[i], n[31 - i]));
            l[i] = max(l[i], n[31 - i]);
            asm volatile("" : "+v"(rest), "+v"(l[i]));         // (in this order: both inputs end here)
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    __builtin_amdgcn_sched_barrier(0);
    meet(std::integral_constant<int, 32>{});
    bitonic_desc<0, 32>(l);
    __builtin_amdgcn_sched_barrier(0);
    meet(std::integral_constant<int, 64>{});
    bitonic_desc<0, 32>(l);
    __builtin_amdgcn_sched_barrier(0);
    meet(std::integral_constant<int, 96>{});
    int t16 = 0x7fffffff, n16 = -1, t32 = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int hi = max(l[i], l[16 + i]), lo = min(l[i], l[16 + i]);
        t16 = min(t16, hi);
        n16 = max(n16, lo);
        t32 = min(t32, lo);
    }
    c.t[0] = t16; c.nx[0] = n16; c.t[1] = t32; c.nx[1] = rest; c.t[2] = 0; c.nx[2] = -1;
    return c;
}

template <int G>
__device__ __forceinline__ Cuts cuts_of(const float (&y)[D], const Trunc &tr) {
    Cuts c;
    if constexpr (G >= 2) {
        constexpr int N = D / G;
        int k[N];
        load_keys<G, 0, N>(y, tr, k, 0);
        oe_sort<0, N - 1>(k);
#pragma unroll
        for (int i = 0; i < 3; ++i) { c.t[i] = k[16 * (i + 1) / G - 1]; c.nx[i] = k[16 * (i + 1) / G]; }
    } else {
        // the 48 largest so far stay sorted; 32 or 16 more come in at a time,
        // sorted, their larger halves against the list's tail (128 keys at
        // once, beside the 128 channels, would not leave two waves per SIMD)
        int l[48], rest = -1;
        {
            int a[32], b[16];
            load_keys<1, 0, 32>(y, tr, a, 0);
            oe_sort<0, 31>(a);
            load_keys<1, 32, 16>(y, tr, b, 0);
            oe_sort<0, 15>(b);
            int m[48];
#pragma unroll
            for (int i = 0; i < 32; ++i) m[i] = a[i];
#pragma unroll
            for (int i = 0; i < 16; ++i) m[32 + i] = b[i];
            oe_merge<0, 63, 1, 48>(m);
#pragma unroll
            for (int i = 0; i < 48; ++i) l[i] = m[i];
        }
        auto round32 = [&](auto first) {
            int n[32], m[48];
            load_keys<1, decltype(first)::value, 32>(y, tr, n, 0);
            oe_sort<0, 31>(n);
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                m[i] = max(l[16 + i], n[31 - i]);
                rest = max(rest, min(l[16 + i], n[31 - i]));
            }
            bitonic_desc<0, 32>(m);
#pragma unroll
            for (int i = 0; i < 16; ++i) m[32 + i] = l[i];
            oe_merge<0, 63, 1, 48>(m);
#pragma unroll
            for (int i = 0; i < 48; ++i) l[i] = m[i];
        };
        __builtin_amdgcn_sched_barrier(0);
        round32(std::integral_constant<int, 48>{});
        __builtin_amdgcn_sched_barrier(0);
        round32(std::integral_constant<int, 80>{});
        __builtin_amdgcn_sched_barrier(0);
        {
            int n[16], m[48];
            load_keys<1, 112, 16>(y, tr, n, 0);
            oe_sort<0, 15>(n);
#pragma unroll
            for (int i = 0; i < 32; ++i) m[i] = l[i];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                m[32 + i] = max(l[32 + i], n[15 - i]);
                rest = max(rest, min(l[32 + i], n[15 - i]));
            }
            bitonic_desc<32, 16>(m);
            oe_merge<0, 63, 1, 48>(m);
            c.t[0] = m[15]; c.nx[0] = m[16]; c.t[1] = m[31]; c.nx[1] = m[32]; c.t[2] = m[47]; c.nx[2] = rest;
        }
    }
    return c;
}

// groups equal to the cut that are kept (r / G groups kept, those above it first)
template <int G, int... I>
__device__ __forceinline__ int above_cut(const float (&y)[D], const Trunc &tr, int t, std::integer_sequence<int, I...>) {
    int n = 0;
    auto add = [&](int k) { asm("v_cmp_gt_i32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, 0, %0, vcc" : "+v"(n) : "v"(k), "v"(t) : "vcc"); };
    (add(group_key<G, I, true>(y, tr)), ...);
    return n;
}

// e where k < t, else 0 (compare and select together: the scheduler would
// otherwise run the compares ahead and spill their results)
__device__ __forceinline__ float below_cut(float e, int k, int t) {
    float o;
    asm("v_cmp_gt_i32 vcc, %2, %1\n\tv_cndmask_b32 %0, 0, %3, vcc" : "=v"(o) : "v"(k), "v"(t), "v"(e) : "vcc");
    return o;
}

// energy of the channels dropped with r kept (cut t; ties: some lane's next
// score equals its cut)
template <int G>
__device__ __forceinline__ float dropped(const float (&y)[D], const Trunc &tr, int r, int t, bool ties) {
    auto energy = [&](auto i, auto side) {
        auto e = [&](int j) { const float x = chan<decltype(side)::value>(y, G * decltype(i)::value + j); return x * x; };
        if constexpr (G == 1) return e(0);
        else if constexpr (G == 2) return e(0) + e(1);
        else return (e(0) + e(1)) + (e(2) + e(3));
    };
    if (!ties) {
        auto leaf = [&](auto i) {
            bound_ahead<decltype(i)::value, 8 / G>();
            return below_cut(energy(i, std::false_type{}), group_key<G, decltype(i)::value>(y, tr), t);
        };
        return leaf_tree<0, D / G>(leaf);
    }
    const int m = r / G - above_cut<G>(y, tr, t, std::make_integer_sequence<int, D / G>{});
    int n = 0;
    auto leaf = [&](auto i) {
        const int k = group_key<G, decltype(i)::value, true>(y, tr);
        const float e = energy(i, std::true_type{});
        const bool eq = k == t, kept = (k > t) | (eq & (n < m));
        n += eq ? 1 : 0;
        __builtin_amdgcn_sched_barrier(0);
        return kept ? 0.0f : e;
    };
    return leaf_tree<0, D / G>(leaf);
}

// the same for 16 and 32 kept at once (cuts t16, t32, no ties): squares, sums
// and scores are shared
template <int G>
__device__ __forceinline__ void dropped_pair(const float (&y)[D], const Trunc &tr, int t16, int t32, float &d16, float &d32) {
    struct Two { float a, b; };
    auto leaf = [&](auto i) {
        constexpr int I = decltype(i)::value;
        bound_ahead<I, 8 / G>();
        auto e = [&](int j) { const float x = y[G * I + j]; return x * x; };
        float s;
        if constexpr (G == 1) s = e(0);
        else if constexpr (G == 2) s = e(0) + e(1);
        else s = (e(0) + e(1)) + (e(2) + e(3));
        const int k = group_key<G, I>(y, tr);
        return Two{below_cut(s, k, t16), below_cut(s, k, t32)};
    };
    auto tree = [&](auto self, auto first, auto n) -> Two {
        constexpr int B = decltype(first)::value, N = decltype(n)::value;
        if constexpr (N == 1) return leaf(first);
        else {
            const Two a = self(self, first, std::integral_constant<int, N / 2>{});
            const Two b = self(self, std::integral_constant<int, B + N / 2>{}, std::integral_constant<int, N / 2>{});
            return Two{a.a + b.a, a.b + b.b};
        }
    };
    const Two t = tree(tree, std::integral_constant<int, 0>{}, std::integral_constant<int, D / G>{});
    d16 = t.a; d32 = t.b;
}

// w <- 2 w + (k >= t)
__device__ __forceinline__ void push_bit(uint32_t &w, int k, int t) {
    asm("v_cmp_ge_i32 vcc, %1, %2\n\tv_addc_co_u32 %0, vcc, %0, %0, vcc" : "+v"(w) : "v"(k), "v"(t) : "vcc");
}
template <int G, int W, int NB, int... I>
__device__ __forceinline__ uint32_t mask_word(const float (&y)[D], const Trunc &tr, int t, std::integer_sequence<int, I...>) {
    uint32_t w = 0u;
    auto one = [&](auto i) {
        bound_ahead<decltype(i)::value, 8>();
        push_bit(w, group_key<G, 32 * W + NB - 1 - decltype(i)::value>(y, tr), t);
    };
    (one(std::integral_constant<int, I>{}), ...);
    return w;
}
template <int G, int W, int NB, int... I>
__device__ __forceinline__ uint32_t mask_word_ties(const float (&y)[D], const Trunc &tr, int t, int m, int &n,
                                                   std::integer_sequence<int, I...>) {
    uint32_t w = 0u;
    auto one = [&](auto i) {
        constexpr int J = decltype(i)::value;
        const int k = group_key<G, 32 * W + J, true>(y, tr);
        const bool eq = k == t, kept = (k > t) | (eq & (n < m));
        n += eq ? 1 : 0;
        w |= kept ? (1u << J) : 0u;
        __builtin_amdgcn_sched_barrier(0);
    };
    (one(std::integral_constant<int, I>{}), ...);
    return w;
}
// bit i of the 128 / G: group i is kept
template <int G>
__device__ __forceinline__ void kept_mask(const float (&y)[D], const Trunc &tr, int r, int t, bool ties, uint32_t (&mw)[4]) {
    using S = std::make_integer_sequence<int, 32>;
    mw[0] = mw[1] = mw[2] = mw[3] = 0u;
    if (!ties) {
        mw[0] = mask_word<G, 0, 32>(y, tr, t, S{});
        if constexpr (G <= 2) mw[1] = mask_word<G, 1, 32>(y, tr, t, S{});
        if constexpr (G == 1) { mw[2] = mask_word<G, 2, 32>(y, tr, t, S{}); mw[3] = mask_word<G, 3, 32>(y, tr, t, S{}); }
        return;
    }
    const int m = r / G - above_cut<G>(y, tr, t, std::make_integer_sequence<int, D / G>{});
    int n = 0;
    mw[0] = mask_word_ties<G, 0, 32>(y, tr, t, m, n, S{});
    if constexpr (G <= 2) mw[1] = mask_word_ties<G, 1, 32>(y, tr, t, m, n, S{});
    if constexpr (G == 1) {
        mw[2] = mask_word_ties<G, 2, 32>(y, tr, t, m, n, S{});
        mw[3] = mask_word_ties<G, 3, 32>(y, tr, t, m, n, S{});
    }
}

// ------------------------------------------------------------------ block means
// Means of the rotated keys over blocks of 16, 8 and 4 tokens (ascending
// adds, then times 1 / B), lane per channel, half of the channels at a time.
// Chains that start at the same token share their first adds.
template <int H>
__device__ __forceinline__ void half_means(const float (&y)[D], EncSmem &sm) {
    const int lane = threadIdx.x & 63;
    wave_fence();
#pragma unroll
    for (int c = 0; c < YH; c += 2) *(float2 *)&sm.yb[lane * YB_STRIDE + c] = make_float2(y[H * YH + c], y[H * YH + c + 1]);
    wave_fence();
    float *m = sm.mean + H * YH + lane;
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
        float v[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) v[t] = sm.yb[(16 * q + t) * YB_STRIDE + lane];
        float a16 = v[0], a8 = 0.0f, a4 = 0.0f;
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            if (t > 0) a16 = a16 + v[t];
            if (t == 8) a8 = v[t];
            if (t > 8) a8 = a8 + v[t];
            if (t == 4 || t == 12) a4 = v[t];
            else if (t >= 4 && t != 8 && (t & 4)) a4 = a4 + v[t];
            if (t == 3) m[(12 + 4 * q) * MEAN_STRIDE] = a16 * 0.25f;
            if (t == 7) { m[(12 + 4 * q + 1) * MEAN_STRIDE] = a4 * 0.25f; m[(4 + 2 * q) * MEAN_STRIDE] = a16 * 0.125f; }
            if (t == 11) m[(12 + 4 * q + 2) * MEAN_STRIDE] = a8 * 0.25f;
            if (t == 15) {
                m[(12 + 4 * q + 3) * MEAN_STRIDE] = a4 * 0.25f;
                m[(4 + 2 * q + 1) * MEAN_STRIDE] = a8 * 0.125f;
                m[q * MEAN_STRIDE] = a16 * 0.0625f;
            }
        }
    }
}

// deviation of the lane's token from its block's mean
__device__ __forceinline__ float block_dev(const float (&y)[D], const EncSmem &sm, int log2b) {
    const float *m = sm.mean + (mean_row0(log2b) + ((threadIdx.x & 63) >> log2b)) * MEAN_STRIDE;
    auto leaf = [&](auto i) {
        constexpr int I = decltype(i)::value;
        bound_ahead<I, 4>();
        const float4 a = *(const float4 *)(m + 4 * I);
        const float d0 = y[4 * I] - a.x, d1 = y[4 * I + 1] - a.y, d2 = y[4 * I + 2] - a.z, d3 = y[4 * I + 3] - a.w;
        return (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
    };
    return leaf_tree<0, D / 4>(leaf);
}

// ------------------------------------------------------------------ packing
// f2h and f2e4m3 on the conversion instructions (equal on every finite fp32)
template <int DT>
__device__ __forceinline__ uint16_t half_of(float f) {
    if constexpr (DT) return __builtin_bit_cast(uint16_t, (__bf16)f);
    else return __builtin_bit_cast(uint16_t, (_Float16)f);
}
template <int DT>
__device__ __forceinline__ uint32_t half2_of(float a, float b) {
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    if constexpr (DT) return __builtin_bit_cast(uint32_t, b2{(__bf16)a, (__bf16)b});
    else return (uint32_t)half_of<0>(a) | ((uint32_t)half_of<0>(b) << 16);
}
__device__ __forceinline__ uint32_t e4m3_of(float f) {
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(__builtin_amdgcn_fmed3f(f, -448.0f, 448.0f), 0.0f, 0, false) & 0xffu;
}

// The kept values of token `lane`, in ascending channel order, to p: every
// channel is stored at the position its kept predecessors give, so a dropped
// one is overwritten by the next (a wave's LDS stores complete in order; the
// row has one slot to spare for those after the last).
template <int G, bool F8, int DT>
__device__ __forceinline__ void compact_row(const float (&y)[D], const uint32_t (&mw)[4], uint8_t *p) {
    constexpr uint32_t VB = F8 ? 1 : 2;
#pragma unroll
    for (int i = 0; i < D / G; ++i) {
        const uint32_t kept = __builtin_amdgcn_ubfe(mw[i >> 5], i & 31, 1);
        if constexpr (F8) {
            uint32_t w = 0u;
#pragma unroll
            for (int e = 0; e < G; ++e) w |= e4m3_of(aside(y[G * i + e])) << (8 * e);
            if constexpr (G == 1) *p = (uint8_t)w;
            else if constexpr (G == 2) *(uint16_t *)p = (uint16_t)w;
            else *(uint32_t *)p = w;
        } else if constexpr (G == 1) {
            *(uint16_t *)p = half_of<DT>(y[i]);
        } else if constexpr (G == 2) {
            *(uint32_t *)p = half2_of<DT>(y[2 * i], y[2 * i + 1]);
        } else if (kept) {                                  // (eight bytes would pass the slot to spare)
            *(uint32_t *)p = half2_of<DT>(y[4 * i], y[4 * i + 1]);
            *(uint32_t *)(p + 4) = half2_of<DT>(y[4 * i + 2], y[4 * i + 3]);
        }
        p += kept * (G * VB);
        if ((i & 3) == 3) __builtin_amdgcn_sched_barrier(0);      // bound the look-ahead
    }
}

// The wave's 64 vectors of one tensor, packed at out (the token records of
// the segment; second: the values' halves of the blocks): bitmaps straight
// from the lanes, kept values staged in st (rows padded by four bytes: an odd
// number of words, so the lanes' stores spread over the banks).
template <int DT>
__device__ __forceinline__ void stage_rows(const float (&y)[D], const Trunc &tr, int r, int log2g, int t, bool ties, bool f8,
                                           uint32_t (&mw)[4], uint8_t *st) {
    uint8_t *row = st + (threadIdx.x & 63) * ((f8 ? r : 2 * r) + 4);
    auto go = [&](auto gc) {
        constexpr int G = decltype(gc)::value;
        kept_mask<G>(y, tr, r, t, ties, mw);
        if (f8) compact_row<G, true, DT>(y, mw, row);
        else compact_row<G, false, DT>(y, mw, row);
    };
    if (log2g == 0) go(std::integral_constant<int, 1>{});
    else if (log2g == 1) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 4>{});
}

__device__ __forceinline__ void write_rows(const uint32_t (&mw)[4], const uint8_t *st, int r, int log2g, int log2b, int T, bool f8,
                                           bool second, uint8_t *out) {
    const int lane = threadIdx.x & 63;
    const int bmb = bm_bytes(log2g, T), vb = f8 ? r : 2 * r, B = 1 << log2b;
    const uint32_t blkb = (uint32_t)(B * 2 * (bmb + vb)), base = second ? (uint32_t)(B * (bmb + vb)) : 0u;
    {
        uint8_t *bm = out + (uint32_t)(lane >> log2b) * blkb + base + (uint32_t)((lane & (B - 1)) * bmb);
        if (T == D) {                                       // 16, 8 or 4 bytes, as aligned as they are long
            if (log2g == 0) *(uint4 *)bm = make_uint4(mw[0], mw[1], mw[2], mw[3]);
            else if (log2g == 1) *(uint2 *)bm = make_uint2(mw[0], mw[1]);
            else *(uint32_t *)bm = mw[0];
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k)                    // T <= 96: at most 12 bytes
                if (k < bmb) bm[k] = (uint8_t)(mw[k >> 2] >> (8 * (k & 3)));
        }
    }
    // the staged rows, a dword per lane and step
    wave_fence();
    const int wpt = vb >> 2;                                // dwords of a token's values: 4, 8, 12, 16 or 24
    const uint32_t inv = 65536u / (uint32_t)wpt + 1u;       // i / wpt = i * inv >> 16 for i < 64 * 24
    for (int k = 0; k < wpt; ++k) {
        const uint32_t i = (uint32_t)(lane + 64 * k), tk = (i * inv) >> 16, w = i - tk * (uint32_t)wpt;
        const uint32_t v = *(const uint32_t *)(st + tk * (uint32_t)(vb + 4) + 4 * w);
        *(uint32_t *)(out + (tk >> log2b) * blkb + base + (uint32_t)(B * bmb) + (tk & (uint32_t)(B - 1)) * (uint32_t)vb + 4 * w) = v;
    }
}

// ------------------------------------------------------------------ block keys
// Four block keys at a time, lane per channel (lane, lane + 64): the r-th
// largest score by a search over its bits, the wave's ballots counting the
// channels at or above the trial value (a group's channels share its score,
// so r channels are r / g groups); the search ends when a trial separates
// exactly r.  Four at once keep the scalar chain of one off the others'.
constexpr int KEYS = 4;

template <int DT>
__device__ __forceinline__ void pack_keys(const EncSmem &sm, int r, int log2g, int log2b, int T, uint8_t *sc) {
    const int lane = threadIdx.x & 63, nb = SEG >> log2b;
    const int bmb = bm_bytes(log2g, T), srec = 2 * r + bmb;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int k0 = 0; k0 < nb; k0 += KEYS) {
        float ylo[KEYS], yhi[KEYS];
        int slo[KEYS], shi[KEYS];
#pragma unroll
        for (int k = 0; k < KEYS; ++k) {
            const float *m = sm.mean + (mean_row0(log2b) + k0 + k) * MEAN_STRIDE;
            ylo[k] = m[lane]; yhi[k] = m[lane + 64];
            float a = fabsf(ylo[k]), b = fabsf(yhi[k]);
            // group sums of adjacent lanes (lane ^ 1, then lane ^ 2: quad permutes)
            if (log2g >= 1) { a = a + dpp_read<0xb1, 0xf>(a); b = b + dpp_read<0xb1, 0xf>(b); }
            if (log2g >= 2) { a = a + dpp_read<0x4e, 0xf>(a); b = b + dpp_read<0x4e, 0xf>(b); }
            slo[k] = lane < T ? __float_as_int(a) : -1;
            shi[k] = lane + 64 < T ? __float_as_int(b) : -1;
        }
        int t[KEYS], cnt[KEYS];
#pragma unroll
        for (int k = 0; k < KEYS; ++k) { t[k] = 0; cnt[k] = T; }
        for (int bit = 30; bit >= 0; --bit) {
            bool open = false;
#pragma unroll
            for (int k = 0; k < KEYS; ++k) {
                const int v = t[k] | (1 << bit);
                const int c = (int)__popcll(__ballot(slo[k] >= v)) + (int)__popcll(__ballot(shi[k] >= v));
                const bool up = cnt[k] != r && c >= r;
                t[k] = up ? v : t[k];
                cnt[k] = up ? c : cnt[k];
                open |= cnt[k] != r;
            }
            if (!open) break;
        }
#pragma unroll
        for (int k = 0; k < KEYS; ++k) {
            uint64_t mlo = __ballot(slo[k] >= t[k]), mhi = __ballot(shi[k] >= t[k]);
            if (cnt[k] != r) {                              // ties at the cut: the lower indices
                const uint64_t elo = __ballot(slo[k] == t[k]), ehi = __ballot(shi[k] == t[k]);
                const int need = r - (int)__popcll(mlo & ~elo) - (int)__popcll(mhi & ~ehi);
                const bool klo = slo[k] > t[k] || (slo[k] == t[k] && (int)__popcll(elo & below) < need);
                const bool khi = shi[k] > t[k] || (shi[k] == t[k] && (int)(__popcll(elo) + __popcll(ehi & below)) < need);
                mlo = __ballot(klo); mhi = __ballot(khi);
            }
            uint8_t *bm_out = sc + (uint32_t)(k0 + k) * (uint32_t)srec, *val_out = bm_out + bmb;
            // truncated bitmaps of 3 or 6 bytes put records at odd bytes: a byte at a time
            auto put16 = [&](int slot, uint16_t h) {
                if (T < D) { val_out[2 * slot] = (uint8_t)h; val_out[2 * slot + 1] = (uint8_t)(h >> 8); }
                else *(uint16_t *)(val_out + 2 * slot) = h;
            };
            if ((mlo >> lane) & 1ull) put16((int)__popcll(mlo & below), half_of<DT>(ylo[k]));
            if ((mhi >> lane) & 1ull) put16((int)__popcll(mlo) + (int)__popcll(mhi & below), half_of<DT>(yhi[k]));
            // group flags in bitmap order: group i's first channel is i g of its half
            uint64_t b0 = mlo, b1 = mhi;
            if (log2g) {
                const int gph = 64 >> log2g, src = (lane % gph) << log2g;
                const bool flag = (lane < 2 * gph) && ((((lane / gph) ? mhi : mlo) >> src) & 1ull);
                b0 = __ballot(flag);
                b1 = 0ull;
            }
            if (T < D) {
                if (lane < bmb) bm_out[lane] = (uint8_t)((lane < 8 ? b0 >> (8 * lane) : b1 >> (8 * (lane - 8))) & 0xffu);
            } else if (lane < (bmb >> 2)) {
                ((uint32_t *)bm_out)[lane] = (uint32_t)((lane < 2 ? b0 : b1) >> (32 * (lane & 1)));
            }
        }
    }
}

// ------------------------------------------------------------------ the kernel
// MODE 0: choose the segment's strategy; 1: pack it at its descriptor's
// offsets; 2: both from one rotation, into the segment's worst-case slot of
// the workspace (slot_tok + slot_sc bytes per (pair, segment)).  With close
// set (modes 0 and 1) the segments are those of each pair's window awaiting
// its rotation, and the input holds that window's tokens from its first one.
template <int MODE, int DT>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_encode(Geom g, const uint16_t *k, const uint16_t *v, int64_t seq_stride, uint8_t *ws, uint32_t slot_tok,
         uint32_t slot_sc, int close) {
    __shared__ __align__(16) EncSmem sm;
    const int p = blockIdx.y;
    const PairMeta *meta = g.meta_of(p);
    int seg = blockIdx.x, win;
    if (close) {
        const int pw = meta->pend;
        if (pw < 0) return;
        const int32_t *wt = g.wtab_of(p);
        seg += wt[pw];
        if (seg >= wt[pw + 1]) return;
        win = pw;
    } else {
        if (seg >= meta->L / SEG) return;
        win = (seg * SEG) / g.W;
    }
    const int which = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);      // 0: keys, 1: values
    Desc *desc = g.desc_of(p) + seg;
    const uint16_t *src = (which ? v : k) + ((uint64_t)p * seq_stride + (uint64_t)blockIdx.x * SEG) * D;
    float y[D];
    if (g.rotated) rotate_rows<DT>(src, g.rot_of(p, win) + which * D * D, which ? (uint8_t *)sm.mean : (uint8_t *)sm.yb, y);
    else plain_rows<DT>(src, y);
    lds_barrier();                                          // both waves are done with their input rows' place
    Trunc tr;
#pragma unroll
    for (int i = 0; i < 4; ++i) tr.m[i] = 32 * i < g.trunc ? 0 : -1;

    // ---- strategy: the first (r, g) in candidate order whose dropped energy
    // is below tau_ch * energy for K and for V
    int r = 0, log2g = 0, log2b = 0;
    const bool known = MODE == 1 || g.force;
    if (MODE == 1) { const Desc d = *desc; r = d.r; log2g = d.log2g; log2b = d.log2b; }
    else if (g.force) { r = g.def_keep; log2g = enc_log2(g.def_group); log2b = enc_log2(g.def_block); }
    if (MODE == 0 && g.force) {
        if (threadIdx.x == 0) { desc->r = (uint8_t)r; desc->log2g = (uint8_t)log2g; desc->log2b = (uint8_t)log2b; desc->flags = 0; }
        return;
    }
    float tot = 0.0f, lim = 0.0f;
    if (!known) {
        auto sq = [&](auto i) { constexpr int I = decltype(i)::value; bound_ahead<I, 8>(); return y[I] * y[I]; };
        tot = tree64(leaf_tree<0, D>(sq));
        lim = g.tau_ch * tot;
        renew(y);
    }
    int cut = 0;                                            // this token's cut under the chosen strategy
    bool ties = false;
    {
        // the levels' cuts, by log2 of the group size; with a level's cuts come
        // the dropped energies of its 16 and 32 kept, those of 48 when asked
        int ct[3][3];
        uint32_t have = 0u, tie_bits = 0u, pass = 0u;       // pass, tie_bits: bits 3 log2g + (r / 16 - 1)
        bool have48 = false;                                // the cut of 48 single channels
        int chosen = 0;
        uint32_t slot = 0u;                                 // the next exchange between the waves
        auto agree = [&](uint32_t own) {                    // the bits that both waves set
            if ((threadIdx.x & 63) == 0) sm.pass[slot][which] = own;
            lds_barrier();
            const uint32_t both = (uint32_t)__builtin_amdgcn_readfirstlane((int)(sm.pass[slot][0] & sm.pass[slot][1]));
            ++slot;
            return both;
        };
#pragma unroll
        for (int i = 0; i < 3; ++i) ct[i][0] = ct[i][1] = ct[i][2] = 0;
#pragma unroll 1
        for (int ci = 0; ci < 9; ++ci) {
            renew(y);
            if (!known) { r = g.keep_cand[ci / 3]; log2g = enc_log2(g.group_cand[ci % 3]); }
            const int ri = r / 16 - 1;
            chosen = 3 * log2g + ri;
            const bool full = log2g == 0 && ri == 2 && !have48;
            if (!((have >> log2g) & 1u) || full) {
                auto level = [&](const Cuts &c, int (&t3)[3]) {
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        t3[i] = c.t[i];
                        if (__ballot(c.t[i] == c.nx[i])) tie_bits |= 1u << (3 * log2g + i);
                    }
                };
                if (full) { level(cuts_of<1>(y, tr), ct[0]); have48 = true; }
                else if (log2g == 0) level(cuts32(y, tr), ct[0]);
                else if (log2g == 1) level(cuts_of<2>(y, tr), ct[1]);
                else level(cuts_of<4>(y, tr), ct[2]);
                if (!known && !((have >> log2g) & 1u)) {
                    renew(y);
                    float d16, d32;
                    auto both = [&](auto gc, const int (&t3)[3]) {
                        constexpr int G = decltype(gc)::value;
                        if ((tie_bits >> (3 * log2g)) & 3u) {
                            d16 = dropped<G>(y, tr, 16, t3[0], true);
                            d32 = dropped<G>(y, tr, 32, t3[1], true);
                        } else dropped_pair<G>(y, tr, t3[0], t3[1], d16, d32);
                    };
                    if (log2g == 0) both(std::integral_constant<int, 1>{}, ct[0]);
                    else if (log2g == 1) both(std::integral_constant<int, 2>{}, ct[1]);
                    else both(std::integral_constant<int, 4>{}, ct[2]);
                    pass |= agree((tree64(d16) < lim ? 1u : 0u) | (tree64(d32) < lim ? 2u : 0u)) << (3 * log2g);
                }
                have |= 1u << log2g;
            }
            if (known || ci == 8) break;                    // the last candidate needs no test
            if (ri == 2) {
                renew(y);
                const bool tie = (tie_bits >> chosen) & 1u;
                float d;
                if (log2g == 0) d = dropped<1>(y, tr, 48, ct[0][2], tie);
                else if (log2g == 1) d = dropped<2>(y, tr, 48, ct[1][2], tie);
                else d = dropped<4>(y, tr, 48, ct[2][2], tie);
                if (agree(tree64(d) < lim ? 1u : 0u)) break;
            } else if ((pass >> chosen) & 1u) {
                break;
            }
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) cut = chosen == i ? ct[i / 3][i % 3] : cut;
        ties = (tie_bits >> chosen) & 1u;
    }

    // ---- first the keys' wave takes the block means, and the first block size
    // whose deviation is below tau_blk * energy (the last candidate needs no
    // test), while the values' wave stages its records; then the keys' wave
    // stages its own over the channels the means came from
    uint32_t mw[4];
    uint8_t *st = which ? sm.vst : (uint8_t *)sm.yb;
#pragma unroll 1
    for (int step = 0; step < 2; ++step) {
        renew(y);
        if (which == step) {
            if (step == 0) {
                half_means<0>(y, sm);
                half_means<1>(y, sm);
                wave_fence();
                if (!known) {
                    const float lb = g.tau_blk * tot;
                    log2b = enc_log2(g.block_cand[2]);
#pragma unroll 1
                    for (int bi = 0; bi < 2; ++bi) {
                        const int l2 = enc_log2(g.block_cand[bi]);
                        const float vb = tree64(block_dev(y, sm, l2));
                        if (vb < lb) { log2b = l2; break; }
                    }
                    log2b = __builtin_amdgcn_readfirstlane(log2b);
                    if (threadIdx.x == 0) sm.log2b = log2b;
                }
            }
        } else if (MODE != 0) {
            stage_rows<DT>(y, tr, r, log2g, cut, ties, g.fp8 != 0, mw, st);
        }
        if (MODE == 0) {
            if (threadIdx.x == 0) { desc->r = (uint8_t)r; desc->log2g = (uint8_t)log2g; desc->log2b = (uint8_t)log2b; desc->flags = 0; }
            return;
        }
        if (step == 0) {
            lds_barrier();                                  // the means and the block size
            if (!known) log2b = __builtin_amdgcn_readfirstlane(sm.log2b);
        }
    }
    uint8_t *tok, *sc;
    if (MODE == 2) {
        if (threadIdx.x == 0) { desc->r = (uint8_t)r; desc->log2g = (uint8_t)log2g; desc->log2b = (uint8_t)log2b; desc->flags = 0; }
        tok = ws + ((uint64_t)p * g.max_desc + seg) * ((uint64_t)slot_tok + slot_sc);
        sc = tok + slot_tok;
    } else {
        tok = g.tok_of(p) + desc->tok_off;
        sc = g.sc_of(p) + desc->sc_off;
    }
    write_rows(mw, st, r, log2g, log2b, g.trunc, g.fp8 != 0, which != 0, tok);
    if (which) pack_keys<DT>(sm, r, log2g, log2b, g.trunc, sc);
}

template <int DT>
hipError_t encode_dt(const Geom &g, int mode, const uint16_t *k, const uint16_t *v, int64_t seq_stride, uint8_t *ws,
                     uint32_t slot_tok, uint32_t slot_sc, int segs, int close, hipStream_t s) {
    const dim3 grid(segs, g.npairs);
    if (mode == 0) hipLaunchKernelGGL((k_encode<0, DT>), grid, dim3(128), 0, s, g, k, v, seq_stride, ws, slot_tok, slot_sc, close);
    else if (mode == 1) hipLaunchKernelGGL((k_encode<1, DT>), grid, dim3(128), 0, s, g, k, v, seq_stride, ws, slot_tok, slot_sc, close);
    else hipLaunchKernelGGL((k_encode<2, DT>), grid, dim3(128), 0, s, g, k, v, seq_stride, ws, slot_tok, slot_sc, close);
    return hipGetLastError();
}

}  // namespace

// every kept count of the strategy set is one the sorting networks deliver
bool encode_fits(const Geom &g) {
    auto ok = [](int r) { return r == 16 || r == 32 || r == 48; };
    return ok(g.keep_cand[0]) && ok(g.keep_cand[1]) && ok(g.keep_cand[2]) && ok(g.def_keep);
}

hipError_t launch_encode(const Geom &g, int mode, const uint16_t *k, const uint16_t *v, int64_t seq_stride, uint8_t *ws,
                         uint32_t slot_tok, uint32_t slot_sc, int segs, int close, hipStream_t s) {
    if (g.dtype) return encode_dt<1>(g, mode, k, v, seq_stride, ws, slot_tok, slot_sc, segs, close, s);
    return encode_dt<0>(g, mode, k, v, seq_stride, ws, slot_tok, slot_sc, segs, close, s);
}

}  // namespace mosaic
