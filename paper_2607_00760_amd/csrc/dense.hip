// dense.hip -- uncompressed split-K decode attention (the "Full" baseline of
// Sec. 6.1) on the same K/V layout the compression pass reads.
//
// One workgroup per (pair, run of 1024-token chunks), four waves that take
// 32-token steps in turn; a log-sum-exp merge of the runs follows.  HBM is the
// bound, so everything else is kept off its way: K rows go from memory
// straight into matrix-core operands (a lane's 16 bytes of a row are 8
// channels of the product's inner dimension), V rows go by direct loads into
// LDS, from where the transposing reads hand them to the second product, and
// both are loaded one step ahead.  The weights take part as three 16-bit parts,
// which hold all 24 bits of the fp32 weight in either type; with up to four
// heads the parts share one product, so the third costs nothing.
// 4 x 32768 tokens, 8 kv heads, bf16 (537 MB): lane-per-token dot products on
// the vector ALU took 200 us (2.7 TB/s); this takes 101 us (5.3 TB/s).
#include "dense_step.h"

namespace mosaic {

namespace {

constexpr int DCHUNK = 1024;              // tokens of the smallest run (and of a partial's share of the workspace)
constexpr int DNWV = 4;
// Chunks are joined into longer runs so that about DRUNS runs remain, at least
// two rounds of the 512 workgroups that the chip holds: about 1024 to 2047 from
// DRUNS chunks on (the division rounds down).  Rounded up, 512 to 1024 remain and
// fill one to two rounds unevenly.  us, 40000 tokens each, bf16, one kv head:
//   sequences      32     40     51     60     70   |  7 of 8 kv heads
//   down        124.0  158.0  188.5  218.4  257.6   |  211.5
//   up          133.3  168.3  184.6  234.2  256.5   |  225.7
constexpr int DRUNS = 1024;

template <int DT, int GP>
__global__ void __launch_bounds__(64 * DNWV) __attribute__((amdgpu_waves_per_eu(2)))
k_dense_split(const uint16_t *q, const uint16_t *k, const uint16_t *v, int hkv, int G, int64_t seq_stride, const int32_t *ctx,
              float scale, float *part, int max_splits, int run) {
    using M8 = typename DMma<DT>::v8;
    constexpr float PS = DT ? 1.0f : 16384.0f;               // weights below fp16's normal range keep their bits
    __shared__ __align__(16) uint8_t vt[DNWV][2][DSTEP * D * 2];
    const int p = blockIdx.y, sp = blockIdx.x, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = ctx[p / hkv];
    const int t0 = sp * run;
    if (t0 >= L) return;
    const int t1 = min(L, t0 + run);
    const uint16_t *kp = k + (uint64_t)p * seq_stride * D, *vp = v + (uint64_t)p * seq_stride * D;
    // q operand: column h < G is head h's query
    M8 qb[4];
    {
        const uint16_t *src = q + ((uint64_t)p * G + min(l16, G - 1)) * D + 8 * q4;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            uint16_t w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = l16 < G ? src[32 * ks + i] : (uint16_t)0;   // (q is 2- or 4-byte aligned)
            __builtin_memcpy(&qb[ks], w, 16);
        }
    }
    float m_run = -INFINITY, l_run = 0.0f;                    // head l16
    df4 acc[8];                                               // [channel tile][row 4 q4 + r]
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc[ct] = df4{0.0f, 0.0f, 0.0f, 0.0f};
    typedef __attribute__((address_space(3))) uint8_t lds_b;
    typedef __attribute__((address_space(1))) const uint8_t gl_b;
    // rows past the context read its last row; their weights are zero
    auto load_k = [&](int t, uint4 (&x)[2][4]) {
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const uint4 *row = (const uint4 *)(kp + (uint64_t)min(t + 16 * n + l16, L - 1) * D) + q4;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) x[n][ks] = row[4 * ks];
        }
    };
    // 16-byte piece c of row r sits at piece c ^ (r % 16): the transposing reads of 16 rows spread over the banks
    auto load_v = [&](int t, int buf) {
#pragma unroll
        for (int i = 0; i < DSTEP / 4; ++i) {
            const int r = 4 * i + (lane >> 4);
            __builtin_amdgcn_global_load_lds((gl_b *)(vp + (uint64_t)min(t + r, L - 1) * D + 8 * ((lane & 15) ^ (r & 15))),
                                             (lds_b *)(&vt[wave][buf][1024 * i]), 16, 0, 0);
        }
    };
    constexpr uint32_t VBUF = DSTEP * D * 2;
    uint32_t va[8];                                           // the transposing reads of each channel tile
    tr_addresses((uint32_t)(uintptr_t)(lds_b *)vt[wave][0], va);
    int t = t0 + DSTEP * wave;
    // one step: the rows of step t in kx and buffer buf, the next step's into kn and the other buffer
    auto step = [&](const uint4 (&kx)[2][4], uint4 (&kn)[2][4], const int buf) {
        const int tn = t + DSTEP * DNWV < t1 ? t + DSTEP * DNWV : t;     // (the last step loads itself again)
        __builtin_amdgcn_sched_barrier(0);
        load_k(tn, kn);
        __builtin_amdgcn_sched_barrier(0);                    // K's loads before V's: the waits below count on it
        load_v(tn, buf ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        float z[2][4];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            df4 a = df4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) a = DMma<DT>::run(__builtin_bit_cast(M8, kx[n][ks]), qb[ks], a);
#pragma unroll
            for (int r = 0; r < 4; ++r) z[n][r] = a[r] * scale;          // token t + 16 n + 4 q4 + r, head l16
        }
        if (t + DSTEP > t1) {
#pragma unroll
            for (int n = 0; n < 2; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (t + 16 * n + 4 * q4 + r >= t1) z[n][r] = -INFINITY;
        }
        dense_accumulate<DT, GP, 3>(z, m_run, l_run, acc, PS, [&] {
            // this step's V rows have landed once only the next step's 8 + 8 loads are out
            asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        }, va, buf * VBUF);
        t += DSTEP * DNWV;
    };
    uint4 k0[2][4], k1[2][4];
    if (t < t1) { load_k(t, k0); load_v(t, 0); }
    while (t < t1) {                                          // (two steps a turn: no copies that would wait on the loads)
        step(k0, k1, 0);
        if (t >= t1) break;
        step(k1, k0, 1);
    }
    // merge the waves (the loads still in flight land before the buffers are reused)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    float *mrg = (float *)vt[wave][0];                         // [16][D + 2]
    if (q4 == 0) { mrg[l16 * (D + 2)] = m_run; mrg[l16 * (D + 2) + 1] = l_run; }
#pragma unroll
    for (int ct = 0; ct < 8; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) mrg[(4 * q4 + r) * (D + 2) + 2 + 16 * ct + l16] = acc[ct][r];
    __syncthreads();
    constexpr int NROW = GP == 4 ? 3 : 2;                      // rows of a head in the accumulator
    constexpr int NT = 64 * DNWV, NE = GP * D / NT;            // outputs of a thread
    __shared__ float mx[GP];                                   // each head's maximum
    float *out = part + ((uint64_t)p * max_splits + sp) * GP * (D + 2);
    bool odd = false;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const int i = tid + e * NT, h = i / D, c = i % D;
        float M = -INFINITY;
        for (int x = 0; x < DNWV; ++x) M = fmaxf(M, ((const float *)vt[x][0])[h * (D + 2)]);
        float A = 0.0f, Ls = 0.0f;
        for (int x = 0; x < DNWV; ++x) {
            const float *mw = (const float *)vt[x][0];
            const float f = (mw[h * (D + 2)] == -INFINITY) ? 0.0f : __expf(mw[h * (D + 2)] - M);
            float a = 0.0f;
#pragma unroll
            for (int n = NROW - 1; n >= 0; --n) a += mw[(h + n * GP) * (D + 2) + 2 + c];
            A += a * (1.0f / PS) * f;
            Ls += mw[h * (D + 2) + 1] * f;
        }
        out[2 * GP + h * D + c] = A;
        if (c == 0) { out[h] = M; out[GP + h] = Ls; mx[h] = M; }
        odd |= h < G && !(fabsf(A) < INFINITY);
    }
    // A weight in parts times an infinite element is an infinity of either sign
    // or NaN, where the weight itself gives the element's infinity: the run's
    // sums again, with whole weights on the vector ALU (rare; about the 200 us
    // that 4 x 32768 tokens took in this form).
    if (!__syncthreads_or(odd)) return;
    float *wt = (float *)&vt[0][0][0];                         // [NT][GP]: a token's weights
    float a[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) a[e] = 0.0f;
#pragma unroll 1
    for (int b = t0; b < t1; b += NT) {
        if (b + tid < t1) {
            const uint4 *row = (const uint4 *)(kp + (uint64_t)(b + tid) * D);
            float z[GP];
#pragma unroll
            for (int h = 0; h < GP; ++h) z[h] = 0.0f;
#pragma unroll 1
            for (int x = 0; x < D / 8; ++x) {
                const uint4 u = row[x];
                const uint32_t w4[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float kv = h2f((uint16_t)((i & 1) ? (w4[i >> 1] >> 16) : w4[i >> 1]), DT);
#pragma unroll
                    for (int h = 0; h < GP; ++h)
                        if (h < G) z[h] = fmaf(h2f(q[((uint64_t)p * G + h) * D + 8 * x + i], DT), kv, z[h]);
                }
            }
#pragma unroll
            for (int h = 0; h < GP; ++h) wt[tid * GP + h] = mx[h] == -INFINITY ? 0.0f : __expf(z[h] * scale - mx[h]);
        }
        __syncthreads();
        const int n = min(NT, t1 - b);
#pragma unroll 1
        for (int t2 = 0; t2 < n; ++t2)
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const int i = tid + e * NT;
                a[e] = fmaf(wt[t2 * GP + i / D], h2f(vp[(uint64_t)(b + t2) * D + i % D], DT), a[e]);
            }
        __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) out[2 * GP + tid + e * NT] = a[e];
}
static_assert(sizeof(float) * 64 * DNWV * 8 <= DNWV * 2 * DSTEP * D * 2, "the weights fit the V buffers");
static_assert(2 * DSTEP * D * 2 >= 16 * (D + 2) * 4, "the waves' merge fits their V buffers");

// grid (pairs, GP * D / 256): one output per thread; the loads of 32 chunks
// are issued together, then merged by online log-sum-exp
template <int GP>
__global__ void __launch_bounds__(256) k_dense_reduce(int hkv, int G, const int32_t *ctx, const float *part,
                                                      int max_splits, int run, float *outp) {
    constexpr int CB = 32;
    const int p = blockIdx.x, i = blockIdx.y * 256 + threadIdx.x, h = i / D;
    const int L = ctx[p / hkv];
    const int ns = (L + run - 1) / run;
    float M = -INFINITY, Ls = 0.0f, A = 0.0f;
    for (int s0 = 0; s0 < ns; s0 += CB) {
        float m[CB], l[CB], a[CB];
#pragma unroll
        for (int e = 0; e < CB; ++e) {
            if (s0 + e < ns) {
                const float *ps = part + ((uint64_t)p * max_splits + s0 + e) * GP * (D + 2);
                m[e] = ps[h];
                l[e] = ps[GP + h];
                a[e] = ps[2 * GP + i];
            }
        }
#pragma unroll
        for (int e = 0; e < CB; ++e) {
            if (s0 + e < ns && m[e] != -INFINITY) {
                const float mn = fmaxf(M, m[e]);
                const float x = (M == -INFINITY) ? 0.0f : __expf(M - mn), y = __expf(m[e] - mn);
                A = A * x + a[e] * y;
                Ls = Ls * x + l[e] * y;
                M = mn;
            }
        }
    }
    if (h < G) outp[(uint64_t)p * G * D + i] = (Ls > 0.0f) ? A / Ls : 0.0f;
}

}  // namespace

size_t dense_part_bytes(int npairs, int G, int max_ctx) {
    const int GP = G <= 4 ? 4 : 8;
    const int ms = max(1, (max_ctx + DCHUNK - 1) / DCHUNK);
    return (size_t)npairs * ms * GP * (D + 2) * sizeof(float);
}

hipError_t launch_dense(const uint16_t *q, const uint16_t *k, const uint16_t *v, float *out, int nseq, int hkv, int G,
                        int dtype, int64_t seq_stride, int max_ctx, const int32_t *ctx, float scale, float *part,
                        hipStream_t s) {
    const int npairs = nseq * hkv;
    const int ms = max(1, (max_ctx + DCHUNK - 1) / DCHUNK);
    const int run = DCHUNK * max(1, (int)((long long)ms * npairs / DRUNS));
    const dim3 grid(ceil_div(max(max_ctx, 1), run), npairs);
    auto split = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(64 * DNWV), 0, s, q, k, v, hkv, G, seq_stride, ctx, scale, part, ms, run);
        return hipGetLastError();
    };
    const hipError_t e = G <= 4 ? (dtype ? split(k_dense_split<1, 4>) : split(k_dense_split<0, 4>))
                                : (dtype ? split(k_dense_split<1, 8>) : split(k_dense_split<0, 8>));
    if (e != hipSuccess) return e;
    if (G <= 4)
        hipLaunchKernelGGL(k_dense_reduce<4>, dim3(npairs, 4 * D / 256), dim3(256), 0, s, hkv, G, ctx, part, ms, run, out);
    else
        hipLaunchKernelGGL(k_dense_reduce<8>, dim3(npairs, 8 * D / 256), dim3(256), 0, s, hkv, G, ctx, part, ms, run, out);
    return hipGetLastError();
}

}  // namespace mosaic
