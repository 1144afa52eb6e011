// topk.h -- token-budget selection of a pair's blocks by one workgroup (Sec.
// 4.2 stage 2), used by the top-k kernel (decode.hip) and by the fused front
// kernel of short contexts (score.hip) (not part of the C ABI).
#pragma once
#include "decode_common.h"

namespace mosaic {

constexpr int TOPK_BINS = 2048;
constexpr int TOPK_KPT_MAX = 32;                           // keys per thread held in registers, at most

// Token-budget selection (Sec. 4.2 stage 2; Sec. 6.1 selects 10 % of tokens):
// blocks are taken in (score desc, block index asc) order while the tokens
// already taken are fewer than the budget.  The last block taken has the
// threshold key T: a radix selection over the range of the keys finds it,
// each pass histogramming the candidates' TOKENS (block sizes) into 2048 bins
// of width 2^s over the keys still in play, so at most three passes narrow
// the range to T.  Every block above T is taken; the blocks equal to T are
// taken in block order while the tokens taken among them are fewer than what
// the budget still needs (one scan of their tokens).  The selected list is
// written in ascending block order (one scan of the taken counts) together
// with each entry's record info, and the list position where each rotation
// window starts.
constexpr int TOPK_MAXW = MAX_WINDOWS;                     // rotation windows tracked in LDS

// first block of each of the first nwl rotation windows (windows past the
// last segment start at nb)
template <int NT>
__device__ __forceinline__ void window_firsts(const Geom &g, int p, int nb, int ndesc, int nwl, int *fbw) {
    const Desc *gd = g.desc_of(p);
    for (int w = threadIdx.x; w < nwl; w += NT) {
        const int s0 = win_first_seg(g, p, w);
        fbw[w] = (s0 < ndesc) ? (int)gd[s0].first_block : nb;
    }
}

// k and the block count after the window starts
__device__ __forceinline__ void window_tail(const Geom &g, int nb, int k, int32_t *wsel) {
    if (threadIdx.x == 0) { wsel[g.nw] = k; wsel[g.nw + 1] = nb; }
}

// A pair's block scores, sizes and record infos: src.score4(i) and size4(i)
// give four from index i, a multiple of 4 (the lanes past the last block read
// the arrays' slack), info(i) one.
struct TopkGlobal {
    const float *sc;
    const uint8_t *bz;
    const uint2 *bi;
    __device__ __forceinline__ TopkGlobal(const WsGeom &ws, int p)
        : sc(ws.score + (uint64_t)p * (ws.score_stride / 4)), bz(ws.bsize + (uint64_t)p * ws.bsize_stride),
          bi(ws.binfo + (uint64_t)p * (ws.binfo_stride / 8)) {}
    __device__ __forceinline__ float4 score4(int i) const { return *(const float4 *)(sc + i); }
    __device__ __forceinline__ uint32_t size4(int i) const { return *(const uint32_t *)(bz + i); }
    __device__ __forceinline__ uint2 info(int i) const { return bi[i]; }
};

// LDS of a single-workgroup selection of NW waves
constexpr int TK_LIST = 64;                                // candidates ranked directly: one per lane
struct TopkSmem {
    uint32_t hist[2 * TOPK_BINS];
    uint32_t mm[32], pk[16], pub[4], sc[2][16];
    uint32_t cnt[4];                                       // candidates listed, passes in turn
    uint32_t key[TK_LIST], tok[TK_LIST];
    int fbw[TOPK_MAXW];
};

// exclusive prefix sum over the 64 NW threads and the total; s: 16 words of
// LDS that nothing else touches before the next barrier
template <int NW>
__device__ __forceinline__ uint32_t block_excl(uint32_t v, uint32_t &tot, uint32_t *s) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint32_t x = wave_scan_add(v);
    if (NW == 1) {
        tot = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
        return x - v;
    }
    if (lane == 63) s[wv] = x;
    lds_barrier();
    const uint32_t y = wave_scan_add(lane < NW ? s[lane] : 0u);
    const uint32_t base = wv ? (uint32_t)__builtin_amdgcn_readlane((int)y, wv - 1) : 0u;
    tot = (uint32_t)__builtin_amdgcn_readlane((int)y, NW - 1);
    return base + x - v;
}

// Up to 64 NW KPT keys: thread t owns the blocks [KPT t, KPT t + KPT); their
// keys and sizes stay in registers and the taken ones are a KPT-bit mask.  A
// radix pass leaves the threshold's bin; when it holds at most 64 blocks (a
// handful, mostly) every wave ranks them itself, a lane each, instead of two
// more passes of three barriers.  Where all blocks equal to the threshold are
// taken (a single one, mostly) no order among them is needed.  Pairs of few
// blocks take few keys per thread, as their time is that of reading the
// unrolled code once.  8 x 131072 tokens 18.2 -> 17.6
// us, 1 x 4117 tokens 12.1 -> 8.6.
template <int KPT, int NW, typename Src>
__device__ __forceinline__ void topk_reg(const Geom &g, const WsGeom &ws, const Src &src, int p, int nb, int ndesc, int budget,
                                         TopkSmem &sm) {
    constexpr int NT = 64 * NW;
    constexpr int BPT = NW == 16 ? 2 : (NW == 4 ? 4 : 8), LB = NW == 16 ? 11 : (NW == 4 ? 10 : 9);
    static_assert(BPT * NT == 1 << LB && (1 << LB) <= TOPK_BINS, "bins of a pass");
    constexpr int BINS = 1 << LB;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int32_t *sel = ws.sel + (uint64_t)p * (ws.sel_stride / 4);
    int32_t *wsel = ws.wsel + (uint64_t)p * (ws.wsel_stride / 4);
    uint2 *sinfo = ws.selinfo + (uint64_t)p * (ws.selinfo_stride / 8);
    const int i0 = min(nb, tid * KPT), i1 = min(nb, i0 + KPT), n_own = i1 - i0;
    const int nwl = min(g.nw, TOPK_MAXW);
    uint32_t kr[KPT];
    uint32_t zr[KPT / 4];                             // log2 block sizes, four per word
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    {
#pragma unroll
        for (int h = 0; h < KPT / 4; ++h) zr[h] = 4 * h < n_own ? src.size4(i0 + 4 * h) : 0u;
        float4 f[KPT / 4];
#pragma unroll
        for (int q = 0; q < KPT / 4; ++q) f[q] = 4 * q < n_own ? src.score4(i0 + 4 * q) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        window_firsts<NT>(g, p, nb, ndesc, nwl, sm.fbw);       // published by the first barrier
        for (int i = tid; i < BINS; i += NT) sm.hist[i] = 0;
        if (tid < 4) sm.cnt[tid] = 0u;
#pragma unroll
        for (int q = 0; q < KPT / 4; ++q) {
            kr[4 * q] = score_key(f[q].x); kr[4 * q + 1] = score_key(f[q].y);
            kr[4 * q + 2] = score_key(f[q].z); kr[4 * q + 3] = score_key(f[q].w);
        }
#pragma unroll
        for (int j = 0; j < KPT; ++j)
            if (j < n_own) { kmin = min(kmin, kr[j]); kmax = max(kmax, kr[j]); }
    }
    // tokens of owned block j: 2^(log2 size)
    auto tok_reg = [&](int j) -> uint32_t { return 1u << ((zr[j >> 2] >> (8 * (j & 3))) & 7u); };
    kmin = ~wave_max_u(~kmin);
    kmax = wave_max_u(kmax);
    if (NW > 1) {
        if (lane == 0) { sm.mm[wv] = kmin; sm.mm[16 + wv] = kmax; }
        lds_barrier();
        kmin = ~wave_max_u(lane < NW ? ~sm.mm[lane] : 0u);
        kmax = wave_max_u(lane < NW ? sm.mm[16 + lane] : 0u);
    } else {
        lds_barrier();
    }
    uint32_t base = kmin, span = kmax - kmin;                     // candidates: [base, base + span]
    uint32_t rem = (uint32_t)budget;                               // tokens still to take
    bool all_eq = false;                                           // every block equal to the threshold is taken
    for (int pass = 0; budget > 0; ++pass) {
        uint32_t *hc = sm.hist + (pass & 1) * TOPK_BINS, *hn = sm.hist + ((pass + 1) & 1) * TOPK_BINS;
        const int bits = 32 - (span ? __builtin_clz(span) : 32);
        const int sh = bits > LB ? bits - LB : 0;                 // (span >> sh) < BINS
#pragma unroll
        for (int j = 0; j < KPT; ++j) {
            const uint32_t d = kr[j] - base;
            if (j < n_own && kr[j] >= base && d <= span) atomicAdd(&hc[d >> sh], tok_reg(j));
        }
        lds_barrier();
        // the bin holding the rem-th token from the top: thread t owns the BPT
        // bins below BINS - BPT t; zeroes the next pass's bins
        {
            uint32_t h[BPT], own = 0u;
            const int b0 = BINS - BPT * (tid + 1);
#pragma unroll
            for (int e = 0; e < BPT; ++e) { h[e] = hc[b0 + e]; own += h[e]; hn[b0 + e] = 0u; }
            uint32_t tot;
            uint32_t above = block_excl<NW>(own, tot, sm.pk);
            if (above < rem && above + own >= rem) {
#pragma unroll
                for (int e = BPT - 1; e >= 0; --e) {
                    if (above < rem && above + h[e] >= rem) { sm.pub[0] = (uint32_t)(b0 + e); sm.pub[1] = rem - above; sm.pub[2] = h[e]; }
                    above += h[e];
                }
            }
            lds_barrier();
        }
        const uint32_t b = sm.pub[0];
        rem = sm.pub[1];
        base += b << sh;
        span = min(span - (b << sh), sh ? ((1u << sh) - 1u) : 0u);
        if (sh == 0) break;                                       // single keys: the threshold is base
        // the candidates of the bin, listed unless their tokens say that they
        // are many; at most 64 of them are ranked here
        if (sm.pub[2] > TK_LIST * 8) continue;
        uint32_t *cnt = sm.cnt + (pass & 3);
#pragma unroll
        for (int j = 0; j < KPT; ++j)
            if (j < n_own && kr[j] >= base && kr[j] - base <= span) {
                const uint32_t at = atomicAdd(cnt, 1u);
                if (at < TK_LIST) { sm.key[at] = kr[j]; sm.tok[at] = tok_reg(j); }
            }
        lds_barrier();
        const int n = (int)__builtin_amdgcn_readfirstlane((int)*cnt);
        if (n <= TK_LIST) {
            const uint32_t k = lane < n ? sm.key[lane] : 0u, t = lane < n ? sm.tok[lane] : 0u;
            uint32_t gt = 0u, ge = 0u;                            // tokens of the keys above, at or above this lane's
            for (int j = 0; j < n; ++j) {
                const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)k, j), tj = (uint32_t)__builtin_amdgcn_readlane((int)t, j);
                gt += kj > k ? tj : 0u;
                ge += kj >= k ? tj : 0u;
            }
            const uint64_t at = __ballot(lane < n && gt < rem && ge >= rem);
            const int l = (int)__builtin_ctzll(at);               // the threshold's lane (never empty: rem tokens are here)
            base = (uint32_t)__builtin_amdgcn_readlane((int)k, l);
            const uint32_t g1 = (uint32_t)__builtin_amdgcn_readlane((int)gt, l), e1 = (uint32_t)__builtin_amdgcn_readlane((int)ge, l);
            rem -= g1;
            // taken in block order while the tokens before are below rem: all
            // of them when no more than one is needed, or when one remains to
            // cross it
            all_eq = __popcll(at) == 1 || e1 - g1 == rem;
            break;
        }
    }
    // T = base; need = tokens the budget still needs among the blocks equal to T
    const uint32_t T = base, need = rem;
    uint32_t tmask = 0, tot = 0u;
    if (budget > 0 && all_eq) {
#pragma unroll
        for (int j = 0; j < KPT; ++j) tmask |= (j < n_own && kr[j] >= T) ? (1u << j) : 0u;
    } else {
        // this thread's tokens equal to T, then the equal tokens before it:
        // taken are the blocks above T, or equal to T while the equal tokens
        // before are below need
        uint32_t v = 0u;
        if (budget > 0) {
#pragma unroll
            for (int j = 0; j < KPT; ++j) v += (j < n_own && kr[j] == T) ? tok_reg(j) : 0u;
        }
        uint32_t acc = block_excl<NW>(v, tot, sm.sc[0]);
        if (budget > 0) {
#pragma unroll
            for (int j = 0; j < KPT; ++j) {
                const bool eq = j < n_own && kr[j] == T;
                const bool t = j < n_own && (kr[j] > T || (eq && acc < need));
                acc += eq ? tok_reg(j) : 0u;
                tmask |= t ? (1u << j) : 0u;
            }
        }
    }
    // the record info of the taken blocks only: all loads issued, then the stores
    uint2 br[KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) br[j] = ((tmask >> j) & 1u) ? src.info(i0 + j) : make_uint2(0u, 0u);
    const uint32_t pos0 = block_excl<NW>((uint32_t)__popc(tmask), tot, sm.sc[1]);   // list position of this thread's first
    const int k = budget > 0 ? (int)tot : 0;               // blocks selected
    uint32_t *tpos = sm.hist, *tmk = sm.hist + 1024;       // (the histograms are no longer needed)
    tpos[tid] = pos0;
    tmk[tid] = tmask;
    lds_barrier();
    // window starts: the position of the first block at or after each
    // start, from the owning thread's first position and taken mask
    for (int w = tid; w < nwl; w += NT) {
        const int f = sm.fbw[w];
        if (f >= nb) { wsel[w] = k; continue; }
        const int t = f / KPT, off = f % KPT;
        wsel[w] = (int)(tpos[t] + (uint32_t)__popc(tmk[t] & ((1u << off) - 1u)));
    }
    window_tail(g, nb, k, wsel);
    uint32_t pos = pos0;
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
        if ((tmask >> j) & 1u) { sel[pos] = i0 + j; sinfo[pos] = br[j]; }
        pos += (tmask >> j) & 1u;
    }
}

// the token budget of pair p: ceil(rho * scoreable tokens), at least one
// token (0 without scoreable blocks)
__device__ __forceinline__ int pair_budget(const Geom &g, int nb, int nf, int prov) {
    const int ntok = nf * SEG + prov * UBUF;
    if (nb <= 0 || ntok <= 0) return 0;
    const long long bb = ((long long)ntok * g.sel_num + g.sel_den - 1) / g.sel_den;
    return (int)(bb < 1 ? 1 : (bb > ntok ? ntok : bb));
}

}  // namespace mosaic
