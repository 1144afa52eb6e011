// score.hip -- block scoring of the decode step (Sec. 4.2, Sec. 5.3).
//
// Lane per block key.  The packed record (bitmap + values) is read straight
// into registers; a fixed, unrolled slot sequence walks the bitmap's set bits
// in ascending order (v_ffbl on the current word), fp32 fused chain over the
// kept channels, max over the GQA group.  These scores decide the selection,
// so their arithmetic order is fixed.
#include "topk.h"

namespace mosaic {

namespace {

// ------------------------------------------------------------------ score
// One walk: acc[h] += q[c][h] * value over the kept channels c, ascending.
// qs + qoff is the [D][GP] fp32 query of the vector's window.  RV is the
// number of kept values when it is a compile-time constant, else 0 and r
// (wave-uniform over the calling lanes) gives it.  The LDS reads of q run SA
// steps ahead of their products (the positions do not depend on q), so a
// step does not wait for its own read.
template <int DT, int GP, int RMAX, int L2G, int RV>
__device__ __forceinline__ void score_walk(const PVec<RMAX> &x, int r, uint32_t qaddr, float (&acc)[GP]) {
    constexpr int GS = 1 << L2G, NWD = 4 >> L2G;
    constexpr uint32_t QB = GP * 4;                           // bytes of q per channel
    constexpr int NS = (RV ? RV : RMAX) / GS;                 // most steps
    constexpr int SA = GS == 1 ? 2 : 0;                       // reads in flight ahead of use
    constexpr int NQ = GS * (GP / 4);                         // 16-byte reads per step
    Walk wk = make_walk<NWD>(x.bw, qaddr, 32u * GS * QB);      // LDS address of group 0 of word k
    const int n = RV ? RV : r;
    floatx4 ring[SA + 1][NQ];
    auto issue = [&](int j) {                                 // j static in the unrolled code
        const uint32_t qc = wk.a + wk.pos() * (GS * QB);
#pragma unroll
        for (int e = 0; e < GS; ++e)
#pragma unroll
            for (int h4 = 0; h4 < GP; h4 += 4)
                ring[j % (SA + 1)][e * (GP / 4) + h4 / 4] = lds_ld<floatx4>(qc + e * QB + h4 * 4);
        wk.template step<NWD>();
    };
#pragma unroll
    for (int j = 0; j < SA; ++j)
        if (j < NS && (RV || j * GS < n)) issue(j);
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        if (RV || k * GS < n) {                               // wave-uniform
            if (k + SA < NS && (RV || (k + SA) * GS < n)) issue(k + SA);
#pragma unroll
            for (int e = 0; e < GS; ++e) {
                const float xv = h2f_t<DT>(half_at(x.v, k * GS + e));
#pragma unroll
                for (int h4 = 0; h4 < GP; h4 += 4) {
                    const floatx4 q4 = ring[k % (SA + 1)][e * (GP / 4) + h4 / 4];
                    acc[h4] = fmaf(q4[0], xv, acc[h4]);
                    acc[h4 + 1] = fmaf(q4[1], xv, acc[h4 + 1]);
                    acc[h4 + 2] = fmaf(q4[2], xv, acc[h4 + 2]);
                    acc[h4 + 3] = fmaf(q4[3], xv, acc[h4 + 3]);
                }
            }
            if ((k & 3) == 3) __builtin_amdgcn_sched_barrier(0);   // bound the look-ahead
        }
    }
}

// FR: every kept count is 16, 32 or 48 (checked on the host), each with its
// own fully unrolled walk; otherwise one walk with a runtime trip count.  The
// two kinds live in different kernels so that the compiler cannot fold the
// fixed walks into the general one.
template <int DT, int GP, int RMAX, int L2G, bool FR>
__device__ __forceinline__ void score_r(const PVec<RMAX> &x, int r, uint32_t qaddr, float (&acc)[GP]) {
    if (FR) {
        if (r == 32) score_walk<DT, GP, RMAX, L2G, 32>(x, r, qaddr, acc);
        else if (r == 16) score_walk<DT, GP, RMAX, L2G, 16>(x, r, qaddr, acc);
        else score_walk<DT, GP, RMAX, L2G, (RMAX >= 48 ? 48 : 16)>(x, r, qaddr, acc);
    } else {
        score_walk<DT, GP, RMAX, L2G, 0>(x, r, qaddr, acc);
    }
}

// One pass per distinct (r, log2g) among the active lanes, so that every walk
// runs with a wave-uniform trip count and no per-step predicate.
template <int DT, int GP, int RMAX, bool FR>
__device__ __forceinline__ void score_any(const PVec<RMAX> &x, int r, int l2g, uint32_t qaddr, float (&acc)[GP]) {
    const int key = (r << 2) | l2g;
    uint64_t todo = __ballot(1);
    while (todo) {
        const int kv = __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(todo));
        const bool mine = key == kv;
        todo &= ~__ballot(mine);
        if (mine) {
            const int rv = kv >> 2;
            if ((kv & 3) == 0) score_r<DT, GP, RMAX, 0, FR>(x, rv, qaddr, acc);
            else if ((kv & 3) == 1) score_r<DT, GP, RMAX, 1, FR>(x, rv, qaddr, acc);
            else score_r<DT, GP, RMAX, 2, FR>(x, rv, qaddr, acc);
        }
    }
}

// grid (ceil(max segments / spw), pairs): a workgroup scores the block keys of
// spw <= SCORE_SEGS consecutive segments, one lane per block key; spw is at
// most the segments of every window but a pair's last (W, or the least a
// window closed by its loss holds), so a workgroup sees at most two windows.
template <int DT, int GP, int RMAX, bool FR>
__global__ void __launch_bounds__(256) k_score(Geom g, WsGeom ws, int spw) {
    __shared__ __align__(16) float qs[2][D * GP];
    __shared__ Desc ds[SCORE_SEGS];
    __shared__ uint8_t b2s[SCORE_SEGS * 16];                 // block (relative) -> segment (relative)
    __shared__ int s_nblk;

    const int p = blockIdx.y, tid = threadIdx.x;
    const PairMeta meta = *g.meta_of(p);
    int nf, prov, nbuf;
    const int ndesc = pair_ndesc(meta, nf, prov, nbuf);
    const int s0 = blockIdx.x * spw;
    if (s0 >= ndesc) return;
    const int ns = min(spw, ndesc - s0);
    const Desc *gd = g.desc_of(p);
    const uint32_t fb0 = gd[s0].first_block;
    bool plain = true;                      // one channel per group, r a multiple of 8 up to 32, aligned records
    bool dense = true;                      // every channel kept (r = D), aligned records
    if (tid < ns) {
        const Desc d = gd[s0 + tid];
        ds[tid] = d;
        const int nb = ((d.flags & 1) ? UBUF : SEG) >> d.log2b;
        const int o = (int)(d.first_block - fb0);
        for (int j = 0; j < nb; ++j) b2s[o + j] = (uint8_t)tid;
        if (tid == ns - 1) s_nblk = o + nb;
        plain = d.log2g == 0 && d.r <= 32 && (d.sc_off & 3u) == 0;
        dense = d.log2g == 0 && d.r == D && (d.sc_off & 15u) == 0;
    }
    // the window of the first segment and the first segment of the next one
    const int w0 = g.rotated ? win_of_seg(g, p, s0) : 0;
    const int nxt = g.rotated ? win_first_seg(g, p, w0 + 1) : 0x7fffffff;
    const int w1 = (s0 + ns - 1 >= nxt) ? w0 + 1 : w0;
    {
        const float4 *src = (const float4 *)(ws.qrot + (uint64_t)p * (ws.qrot_stride / 4));
        float4 *d0 = (float4 *)qs[0], *d1 = (float4 *)qs[1];
        for (int i = tid; i < D * GP / 4; i += 256) {
            const float4 x0 = src[(uint64_t)w0 * D * GP / 4 + i], x1 = src[(uint64_t)w1 * D * GP / 4 + i];
            d0[i] = x0;
            d1[i] = x1;
        }
    }
    plain = __syncthreads_and(plain);
    if (RMAX >= D) dense = __syncthreads_and(dense);
    const int nblk = s_nblk;
    float *out = ws.score + (uint64_t)p * (ws.score_stride / 4);
    uint2 *binfo = ws.binfo + (uint64_t)p * (ws.binfo_stride / 8);
    uint8_t *bsize = ws.bsize + (uint64_t)p * ws.bsize_stride;
    // a block's token-record offset and strategy (what the selection hands to the attention)
    auto info_of = [&](const Desc &d, int j) {
        return blk_info(d.tok_off + (uint32_t)(j << d.log2b) * (uint32_t)(2 * tok_vec_bytes(d.r, d.log2g, g.trunc, g.fp8)),
                        d.r, d.log2g, d.log2b);
    };
    const uint8_t *sc = g.sc_of(p);
    if constexpr (RMAX >= D) {
        if (dense) {
            // every channel kept: the values are the dense key in channel
            // order; the same ascending fp32 chain reads q row by row (one
            // address for the whole wave)
            for (int b0 = 0; b0 < nblk; b0 += 256) {
                const int b = b0 + tid;
                const bool valid = b < nblk;
                const int i = valid ? b2s[b] : 0;
                const Desc d = ds[i];
                const int j = b - (int)(d.first_block - fb0);
                const uint8_t *rec = valid ? sc + d.sc_off + (uint32_t)j * (uint32_t)vec_bytes(D, 0, g.trunc) : sc;
                const uint4 *v4 = (const uint4 *)(rec + 16);
                uint4 t[D / 8];
#pragma unroll
                for (int k = 0; k < D / 8; ++k) t[k] = v4[k];
                const uint32_t qa = lds_addr(qs) + ((s0 + i >= nxt) ? D * GP * 4 : 0);
                float acc[GP];
#pragma unroll
                for (int h = 0; h < GP; ++h) acc[h] = 0.0f;
#pragma unroll
                for (int k = 0; k < D / 8; ++k) {
                    const uint32_t w4[4] = {t[k].x, t[k].y, t[k].z, t[k].w};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float xv = h2f_t<DT>((e & 1) ? (w4[e >> 1] >> 16) : (w4[e >> 1] & 0xffffu));
#pragma unroll
                        for (int h4 = 0; h4 < GP; h4 += 4) {
                            const floatx4 q4v = lds_ld<floatx4>(qa + (uint32_t)(((8 * k + e) * GP + h4) * 4));
                            acc[h4] = fmaf(q4v[0], xv, acc[h4]);
                            acc[h4 + 1] = fmaf(q4v[1], xv, acc[h4 + 1]);
                            acc[h4 + 2] = fmaf(q4v[2], xv, acc[h4 + 2]);
                            acc[h4 + 3] = fmaf(q4v[3], xv, acc[h4 + 3]);
                        }
                    }
                }
                float best = acc[0];
#pragma unroll
                for (int h = 1; h < GP; ++h)
                    if (h < g.G) best = fmaxf(best, acc[h]);
                if (__float_as_uint(best) == 0x80000000u) best = 0.0f;
                if (valid) {
                    out[d.first_block + j] = best;
                    binfo[d.first_block + j] = info_of(d, j);
                    bsize[d.first_block + j] = d.log2b;
                }
            }
            return;
        }
    }
    if (plain) {
        // one channel per group and at most 32 values: a 16-byte bitmap and
        // four fixed 16-byte value loads at any 4-byte aligned record, and the
        // next key's record is loaded while the current one is scored (one
        // load form, so no join waits on it)
        auto where = [&](int b, int &i, int &j, int &r) {
            const bool valid = b < nblk;
            i = valid ? b2s[b] : 0;
            const Desc d = ds[i];
            j = b - (int)(d.first_block - fb0);
            r = valid ? d.r : 0;
            return valid ? sc + d.sc_off + (uint32_t)j * (uint32_t)vec_bytes(d.r, 0, g.trunc) : sc;
        };
        const int bmb = bm_bytes(0, g.trunc);
        int i, j, r;
        const uint8_t *rec = where(tid, i, j, r);
        PVec<RMAX> x;
        load_pvec<RMAX, 1, false, 4>(x, rec, rec + bmb, 32, true);
        for (int b0 = 0; b0 < nblk; b0 += 256) {
            int in, jn, rn;
            const uint8_t *recn = where(b0 + 256 + tid, in, jn, rn);
            PVec<RMAX> xn;
            __builtin_amdgcn_sched_barrier(0);
            load_pvec<RMAX, 1, false, 4>(xn, recn, recn + bmb, 32, true);
            __builtin_amdgcn_sched_barrier(0);
            if (g.trunc < D) mask_words(x.bw, g.trunc);       // a truncated bitmap's bytes past T bits are values
            const uint32_t qoff = (s0 + i >= nxt) ? D * GP * 4 : 0;
            float acc[GP];
#pragma unroll
            for (int h = 0; h < GP; ++h) acc[h] = 0.0f;
            score_any<DT, GP, RMAX, FR>(x, r, 0, lds_addr(qs) + qoff, acc);
            float best = acc[0];
#pragma unroll
            for (int h = 1; h < GP; ++h)
                if (h < g.G) best = fmaxf(best, acc[h]);
            if (__float_as_uint(best) == 0x80000000u) best = 0.0f;
            if (b0 + tid < nblk) {
                const uint32_t fb = ds[i].first_block;
                out[fb + j] = best;
                binfo[fb + j] = info_of(ds[i], j);
                bsize[fb + j] = ds[i].log2b;
            }
            x = xn; i = in; j = jn; r = rn;
        }
        return;
    }
    for (int b0 = 0; b0 < nblk; b0 += 256) {
        const int b = b0 + tid;
        const bool valid = b < nblk;
        const int i = valid ? b2s[b] : 0;
        const Desc d = ds[i];
        const int j = b - (int)(d.first_block - fb0);
        const int r = valid ? d.r : 0, l2g = d.log2g;
        const uint8_t *rec = valid ? sc + d.sc_off + (uint32_t)j * (uint32_t)vec_bytes(r, l2g, g.trunc) : sc;
        const uint32_t qoff = (s0 + i >= nxt) ? D * GP * 4 : 0;
        const bool a16 = __all(!valid || (l2g == 0 && ((uintptr_t)rec & 15u) == 0 && g.trunc == D));
        PVec<RMAX> x;
        load_pvec<RMAX, -1, true>(x, rec, rec + bm_bytes(l2g, g.trunc), wave_max_i(r), a16);
        if (g.trunc < D) mask_words(x.bw, g.trunc >> l2g);
        float acc[GP];
#pragma unroll
        for (int h = 0; h < GP; ++h) acc[h] = 0.0f;
        score_any<DT, GP, RMAX, FR>(x, r, l2g, lds_addr(qs) + qoff, acc);
        float best = acc[0];
#pragma unroll
        for (int h = 1; h < GP; ++h)
            if (h < g.G) best = fmaxf(best, acc[h]);
        if (__float_as_uint(best) == 0x80000000u) best = 0.0f;
        if (valid) {
            out[d.first_block + j] = best;
            binfo[d.first_block + j] = info_of(d, j);
            bsize[d.first_block + j] = d.log2b;
        }
    }
}

// ------------------------------------------------------------------ short contexts
// grid (pairs): query rotation, scores and selection of a pair of one rotation
// window and at most FRONT_BLOCKS blocks, by one workgroup.  As kernels of
// their own the three take 5 us each before their work counts (launch, code
// fetch, the round trip through memory); here the scores stay in LDS for the
// selection.  What the attention and a caller's inspection read is written as
// the separate kernels write it.  1 x 4117 tokens, 8 kv heads: 4.9 + 8.2 + 8.6
// us apart, 18.0 together (8 requests of 1000 tokens: 20 and 13.8).
constexpr int FRONT_SEGS = FRONT_BLOCKS / 4 + 2;

struct TopkLds {
    const float *sc;
    const uint8_t *bz;
    const uint2 *bi;
    __device__ __forceinline__ float4 score4(int i) const { return *(const float4 *)(sc + i); }
    __device__ __forceinline__ uint32_t size4(int i) const { return *(const uint32_t *)(bz + i); }
    __device__ __forceinline__ uint2 info(int i) const { return bi[i]; }
};

template <int DT, int GP>
__global__ void __launch_bounds__(1024) k_front(Geom g, WsGeom ws, const uint16_t *q) {
    __shared__ float qraw[8][D + 4];
    __shared__ __align__(16) float qs[D * GP];
    __shared__ Desc ds[FRONT_SEGS];
    __shared__ uint16_t b2s[FRONT_BLOCKS];                   // block -> segment
    __shared__ __align__(16) float ssc[FRONT_BLOCKS];
    __shared__ __align__(16) uint8_t sbz[FRONT_BLOCKS];
    __shared__ uint2 sbi[FRONT_BLOCKS];
    __shared__ TopkSmem sm;
    const int p = blockIdx.x, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q4 = lane >> 4, G = g.G;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // R_k^T[4 i + q4][j] for the rotation's eight waves (16 output channels each)
    float r[D / 4];
    const int j = 16 * wave + l16;
    const bool rot = g.rotated && wave < D / 16;
    if (rot) {
        const float *src = g.rot_of(p, 0) + q4 * D + j;
#pragma unroll
        for (int i = 0; i < D / 4; ++i) r[i] = src[4 * i * D];
    }
    const PairMeta meta = *g.meta_of(p);
    if (tid < 8 * D) qraw[tid / D][tid % D] = tid < G * D ? h2f(q[(uint64_t)p * G * D + tid], g.dtype) : 0.0f;
    int nf, prov, nbuf;
    // (the host admits no more: a captured call replayed on a cache that grew
    // since stays inside the arrays)
    const int ndesc = min(pair_ndesc(meta, nf, prov, nbuf), FRONT_SEGS);
    if (tid < ndesc) {
        const Desc d = g.desc_of(p)[tid];
        ds[tid] = d;
        const int nb = ((d.flags & 1) ? UBUF : SEG) >> d.log2b;
        for (int x = 0; x < nb; ++x) b2s[min((int)d.first_block + x, FRONT_BLOCKS - 1)] = (uint16_t)tid;
    }
    __syncthreads();
    const int nblk = ndesc > 0 ? min((int)ds[ndesc - 1].first_block +
                                     (((ds[ndesc - 1].flags & 1) ? UBUF : SEG) >> ds[ndesc - 1].log2b), FRONT_BLOCKS) : 0;
    if (wave < D / 16) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        f4 acc = f4{0.0f, 0.0f, 0.0f, 0.0f};                 // heads 4 q4 .. 4 q4 + 3 of channel j
        if (rot) {                                           // (the fp32 fused chain, as in the rotation kernel)
            const float *qh = &qraw[l16 & 7][q4];
#pragma unroll
            for (int i = 0; i < D / 4; ++i)
                acc = __builtin_amdgcn_mfma_f32_16x16x4f32(l16 < 8 ? qh[4 * i] : 0.0f, r[i], acc, 0, 0, 0);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = qraw[(4 * q4 + e) & 7][j];
        }
        if (4 * q4 < GP) {
            *(f4 *)&qs[j * GP + 4 * q4] = acc;
            *(f4 *)(ws.qrot + (uint64_t)p * (ws.qrot_stride / 4) + (uint64_t)j * GP + 4 * q4) = acc;
        }
    }
    __syncthreads();
    float *out = ws.score + (uint64_t)p * (ws.score_stride / 4);
    uint2 *binfo = ws.binfo + (uint64_t)p * (ws.binfo_stride / 8);
    uint8_t *bsize = ws.bsize + (uint64_t)p * ws.bsize_stride;
    const uint8_t *sc = g.sc_of(p);
    for (int b0 = 0; b0 < nblk; b0 += 1024) {
        const int b = b0 + tid;
        const bool valid = b < nblk;
        if (__ballot(valid) == 0ull) break;                  // (wave-uniform; no barrier inside the loop)
        const Desc d = ds[valid ? b2s[b] : 0];
        const int x0 = b - (int)d.first_block;
        const int rk = valid ? d.r : 0, l2g = d.log2g;
        const uint8_t *rec = valid ? sc + d.sc_off + (uint32_t)x0 * (uint32_t)vec_bytes(rk, l2g, g.trunc) : sc;
        // whole 16-byte granules wherever bitmap and values are 4-byte aligned (what
        // lies past a record is read inside the arena's slack and never used)
        const int bmb = valid ? bm_bytes(l2g, g.trunc) : 0;
        PVec<48> x;
        if (__all((((uintptr_t)rec | (uintptr_t)bmb) & 3u) == 0)) load_pvec<48, 1, false, 6>(x, rec, rec + bmb, 48, true);
        else load_pvec<48, 0, true>(x, rec, rec + bmb, wave_max_i(rk), false);
        if (g.trunc < D) mask_words(x.bw, g.trunc >> l2g);
        float acc[GP];
#pragma unroll
        for (int h = 0; h < GP; ++h) acc[h] = 0.0f;
        score_any<DT, GP, 48, true>(x, rk, l2g, lds_addr(qs), acc);
        float best = acc[0];
#pragma unroll
        for (int h = 1; h < GP; ++h)
            if (h < G) best = fmaxf(best, acc[h]);
        if (__float_as_uint(best) == 0x80000000u) best = 0.0f;
        if (valid) {
            const uint2 info = blk_info(d.tok_off + (uint32_t)(x0 << d.log2b) *
                                        (uint32_t)(2 * tok_vec_bytes(d.r, d.log2g, g.trunc, g.fp8)), d.r, d.log2g, d.log2b);
            out[b] = best; ssc[b] = best;
            binfo[b] = info; sbi[b] = info;
            bsize[b] = d.log2b; sbz[b] = d.log2b;
        }
    }
    __syncthreads();
    const int budget = pair_budget(g, nblk, nf, prov);
    auto on = [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        if (threadIdx.x >= 64 * NW) return;                 // (an ended wave counts at no barrier)
        topk_reg<4, NW>(g, ws, TopkLds{ssc, sbz, sbi}, p, nblk, ndesc, budget, sm);
    };
    if (nblk <= 256) on(IntC<1>{});
    else if (nblk <= 1024) on(IntC<4>{});
    else on(IntC<16>{});
}

template <int DT, int GP>
hipError_t front_dt(const Geom &g, const WsGeom &w, const uint16_t *q, hipStream_t s) {
    hipLaunchKernelGGL((k_front<DT, GP>), dim3(g.npairs), dim3(1024), 0, s, g, w, q);
    return hipGetLastError();
}

template <int DT, int GP>
hipError_t score_dt(const Geom &g, const WsGeom &w, int max_desc_used, bool fixed, bool small, hipStream_t s) {
    // as many segments per workgroup as leave about 1024 workgroups (the chip
    // holds as many), from 8 (64 keys of 8 tokens: a wave) to SCORE_SEGS: one
    // 4096-token sequence of 8 kv heads ran on 8 workgroups of 1024 keys
    // (13.5 us), now on 64 (8.2 us); 4 x 32768 tokens 16.2 -> 10.6 us
    int spw = SCORE_SEGS;
    while (spw > 8 && (long long)ceil_div(max_desc_used, spw) * g.npairs < 1024) spw /= 2;
    spw = max(1, min(spw, (g.dyn ? g.min_win : g.W) / SEG));
    const dim3 grid(ceil_div(max_desc_used, spw), g.npairs);
    if (fixed) hipLaunchKernelGGL((k_score<DT, GP, 48, true>), grid, dim3(256), 0, s, g, w, spw);
    else if (small) hipLaunchKernelGGL((k_score<DT, GP, 48, false>), grid, dim3(256), 0, s, g, w, spw);
    else hipLaunchKernelGGL((k_score<DT, GP, 128, false>), grid, dim3(256), 0, s, g, w, spw);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_front(const Geom &g, const WsGeom &w, const uint16_t *q, hipStream_t s) {
    if (g.dtype) return g.GP == 4 ? front_dt<1, 4>(g, w, q, s) : front_dt<1, 8>(g, w, q, s);
    return g.GP == 4 ? front_dt<0, 4>(g, w, q, s) : front_dt<0, 8>(g, w, q, s);
}

hipError_t launch_score(const Geom &g, const WsGeom &w, int max_desc_used, bool fixed, bool small, hipStream_t s) {
    if (g.dtype) return g.GP == 4 ? score_dt<1, 4>(g, w, max_desc_used, fixed, small, s) : score_dt<1, 8>(g, w, max_desc_used, fixed, small, s);
    return g.GP == 4 ? score_dt<0, 4>(g, w, max_desc_used, fixed, small, s) : score_dt<0, 8>(g, w, max_desc_used, fixed, small, s);
}

}  // namespace mosaic
