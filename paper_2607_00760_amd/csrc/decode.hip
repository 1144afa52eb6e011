// decode.hip -- gfx950 kernels of MosaicKV's decode step (PackedAttention,
// Sec. 5.3; stage-2 dynamic sequence compression, Sec. 4.2).
//
//   qrot   : q . R_k^T once per (pair, window) -- the rotation is merged into
//            the single query vector instead of un-rotating the cache; every
//            output is one fp32 fused chain over the input channels.
//   score  : one fp32 score per block key (score.hip).
//   topk   : exact selection of the k-th largest score key: passes over the
//            range [min, max] of the keys still in play, 2048 bins each, so
//            the bins follow the keys that are present (at most three passes
//            reach a single key), then an ordered compaction that breaks ties
//            by the lowest block index.  Up to 32768 blocks per pair the keys
//            stay in registers (4 to 32 per thread, one workgroup per pair);
//            scans and reductions use lane shifts inside the wave.  Longer
//            pairs are spread over workgroups of 4096 blocks, one kernel per
//            phase.
//   attn   : split-K attention over the selected list and the update buffer
//            (attn.h).
//   combine: log-sum-exp merge of every split of a pair into the output.
#include "topk.h"

namespace mosaic {

namespace {

// ------------------------------------------------------------------ qrot
// grid (windows * 2, pairs), 256 threads: a wave produces 16 output channels of
// every query head of one (pair, window) as a chain of fp32 matrix products,
// whose four products each add in ascending k, one rounding per term: bit for
// bit the fp32 fused chain over the input channels.  R_k^T goes from memory
// straight into operands, all loads in flight at once: no staging and a third
// of the code (the kernel's 5 us are those of any short kernel).
constexpr int QROT_COLS = 64;

__global__ void __launch_bounds__(256) k_qrot(Geom g, WsGeom ws, const uint16_t *q) {
    __shared__ float qs[8][D + 4];                         // rows 4 banks apart
    constexpr int NCG = D / QROT_COLS;
    const int w = blockIdx.x / NCG, tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, q4 = lane >> 4;
    const int j = (blockIdx.x % NCG) * QROT_COLS + 16 * (tid >> 6) + l16;      // this lane's output channel
    const int p = blockIdx.y, G = g.G;
    if (ws.tkx && blockIdx.x == 0) {        // the multi-workgroup top-k's histograms of this call
        uint32_t *h = ws.tkx + (uint64_t)p * (ws.tkx_stride / 4);
        for (int i = tid; i < 3 * 2048; i += 256) h[i] = 0u;
    }
    float r[D / 4];                                        // R_k^T[4 i + q4][j]
    if (g.rotated) {
        const float *src = g.rot_of(p, w) + q4 * D + j;
#pragma unroll
        for (int i = 0; i < D / 4; ++i) r[i] = src[4 * i * D];
    }
    for (int i = tid; i < 8 * D; i += 256) qs[i / D][i % D] = i < G * D ? h2f(q[(uint64_t)p * G * D + i], g.dtype) : 0.0f;
    __syncthreads();
    typedef float f4 __attribute__((ext_vector_type(4)));
    f4 acc = f4{0.0f, 0.0f, 0.0f, 0.0f};                   // heads 4 q4 .. 4 q4 + 3 of channel j
    if (g.rotated) {
        const float *qh = &qs[l16 & 7][q4];
#pragma unroll
        for (int i = 0; i < D / 4; ++i) {
            const float a = l16 < 8 ? qh[4 * i] : 0.0f;
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, r[i], acc, 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] = qs[(4 * q4 + e) & 7][j];
    }
    if (4 * q4 < g.GP) *(f4 *)(ws.qrot + (uint64_t)p * (ws.qrot_stride / 4) + ((uint64_t)w * D + j) * g.GP + 4 * q4) = acc;
}

// ------------------------------------------------------------------ topk
// one workgroup per pair, for calls whose pairs hold at most 32 K blocks
// (longer ones take the multi-workgroup kernels below): the fewest keys per
// thread that hold the pair's blocks
__global__ void __launch_bounds__(1024) k_topk(Geom g, WsGeom ws) {
    __shared__ TopkSmem sm;
    const int p = blockIdx.x;
    const PairMeta meta = *g.meta_of(p);
    const int nb = pair_nblocks(g, p, meta);
    int nf, prov, nbuf;
    const int ndesc = pair_ndesc(meta, nf, prov, nbuf);
    const int budget = pair_budget(g, nb, nf, prov);
    auto on = [&](auto kpt, auto nw) {
        constexpr int NW = decltype(nw)::value;
        if (threadIdx.x >= 64 * NW) return;                 // (an ended wave counts at no barrier)
        topk_reg<decltype(kpt)::value, NW>(g, ws, TopkGlobal(ws, p), p, min(nb, 64 * NW * decltype(kpt)::value), ndesc, budget, sm);
    };
    if (nb <= 256) on(IntC<4>{}, IntC<1>{});
    else if (nb <= 1024) on(IntC<4>{}, IntC<4>{});
    else if (nb <= 4096) on(IntC<4>{}, IntC<16>{});
    else if (nb <= 8192) on(IntC<8>{}, IntC<16>{});
    else if (nb <= 16384) on(IntC<16>{}, IntC<16>{});
    else on(IntC<TOPK_KPT_MAX>{}, IntC<16>{});
}

// ------------------------------------------------------------------ top-k over many workgroups
// sum of s[0 .. n) for n <= 64 (wave-uniform): one read per lane, then the
// lane shifts and the last lane's total (no chain of dependent LDS reads)
__device__ __forceinline__ uint32_t sum_below(const uint32_t *s, int n) {
    const int lane = threadIdx.x & 63;
    const uint32_t x = lane < n ? s[lane] : 0u;
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(x), 63);
}

// exclusive prefix sums over the 1024 threads of the block of N values per
// thread, and their block totals; s: 16 N words of LDS
template <int N>
__device__ __forceinline__ void block_excl_scan_1024(uint32_t (&v)[N], uint32_t (&tot)[N], uint32_t *s) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint32_t x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        x[i] = wave_scan_add(v[i]);
        if (lane == 63) s[16 * i + wv] = x[i];
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t y = wave_scan_add(lane < 16 ? s[16 * i + lane] : 0u);   // inclusive over the waves
        const uint32_t base = wv ? (uint32_t)__builtin_amdgcn_readlane((int)y, wv - 1) : 0u;
        tot[i] = (uint32_t)__builtin_amdgcn_readlane((int)y, 15);
        v[i] = base + x[i] - v[i];
    }
    lds_barrier();
}

// The bin holding the rem-th token from the top of a filled histogram hc
// (2048 bins of width 2^sh over [base, base + span]); zeroes hn for the next
// pass, narrows base / span to that bin and rem to the tokens still needed
// inside it.  True when the bins were single keys (the threshold is base).
__device__ __forceinline__ bool radix_pick(const uint32_t *hc, uint32_t *hn, uint32_t *sbuf, int sh, uint32_t &base,
                                           uint32_t &span, uint32_t &rem) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // bins from the top: thread t owns bins 2047 - 2t and 2046 - 2t
    const uint32_t h0 = hc[TOPK_BINS - 1 - 2 * tid], h1 = hc[TOPK_BINS - 2 - 2 * tid];
    hn[2 * tid] = 0;
    hn[2 * tid + 1] = 0;
    const uint32_t x = wave_scan_add(h0 + h1);
    if (lane == 63) sbuf[wv] = x;
    lds_barrier();
    uint32_t above = x - (h0 + h1);
    above += sum_below(sbuf, wv);
    if (above < rem && above + h0 + h1 >= rem) {
        if (above + h0 >= rem) { sbuf[32] = TOPK_BINS - 1 - 2 * tid; sbuf[33] = rem - above; }
        else { sbuf[32] = TOPK_BINS - 2 - 2 * tid; sbuf[33] = rem - above - h0; }
    }
    lds_barrier();
    const uint32_t b = sbuf[32];
    rem = sbuf[33];
    base += b << sh;
    const uint32_t width = sh ? ((1u << sh) - 1u) : 0u;
    span = min(span - (b << sh), width);
    return sh == 0;
}

// four consecutive keys and their log2 block sizes from index i (a multiple
// of 4 below nb; the lanes past nb read the rest of the arrays' slack)
struct Key4 {
    uint32_t k[4];
    uint32_t z;                                             // four log2 sizes, one per byte
    __device__ __forceinline__ uint32_t tok(int e) const { return 1u << ((z >> (8 * e)) & 7u); }
};
__device__ __forceinline__ Key4 load_key4(const float *sc, const uint8_t *bz, int i) {
    const float4 f = *(const float4 *)(sc + i);
    Key4 r;
    r.k[0] = score_key(f.x); r.k[1] = score_key(f.y); r.k[2] = score_key(f.z); r.k[3] = score_key(f.w);
    r.z = *(const uint32_t *)(bz + i);
    return r;
}

// Calls whose pairs can hold more than 32 K blocks: the same token-budget
// selection, spread over workgroups of TKM_CHUNK consecutive blocks of a pair
// and one kernel per phase, so that a long pair's keys are read by dozens of
// CUs instead of one.  Three radix passes of 11, 11 and 10 bits over the
// key: kernel k first takes the pick of pass k - 1 from the pair's histogram
// of that pass (every workgroup the same, workgroup 0 records the state),
// then adds its chunk's candidates' tokens to the pair's histogram of pass k
// (per-chunk LDS bins, then integer atomics: exact in any order).  After the
// last pick (threshold T, tokens still needed at T) one kernel sums the
// tokens equal to T per chunk, the next counts each chunk's taken blocks
// (blocks above T, and blocks equal to T while the equal tokens before them,
// over the chunks before and the block order inside, are below the need), and
// the last writes the list in block order and the windows' starts.  Chunk
// prefixes are sums over the chunks before (a few dozen).
// Per-pair state (WsGeom::tkx): hist[3][2048] | TkmHdr[4] | eq[nch] | tk[nch];
// the three histograms are zeroed by k_qrot earlier in the same call.
constexpr int TKM_CHUNK = 4096;                            // blocks per workgroup: 1024 threads x 4

struct TkmHdr { uint32_t base, span, rem, done; };          // radix state after each pick

__device__ __forceinline__ uint32_t *tkm_of(const WsGeom &ws, int p) { return ws.tkx + (uint64_t)p * (ws.tkx_stride / 4); }

// this workgroup's view of pair p: blocks, budget, its chunk's keys (four
// consecutive per thread) and the radix state after `npicks` picks
struct TkmCtx {
    int nb, ndesc, budget, i0, n_own;
    Key4 x;
    uint32_t *st;
    __device__ __forceinline__ bool in(int e) const { return e < n_own; }
};

__device__ __forceinline__ bool tkm_setup(const Geom &g, const WsGeom &ws, int p, int c, TkmCtx &t) {
    const PairMeta meta = *g.meta_of(p);
    int nf, prov, nbuf;
    t.ndesc = pair_ndesc(meta, nf, prov, nbuf);
    t.nb = pair_nblocks(g, p, meta);
    t.budget = pair_budget(g, t.nb, nf, prov);
    t.st = tkm_of(ws, p);
    t.i0 = c * TKM_CHUNK + 4 * (int)threadIdx.x;
    t.n_own = max(0, min(4, t.nb - t.i0));
    const float *sc = ws.score + (uint64_t)p * (ws.score_stride / 4);
    const uint8_t *bz = ws.bsize + (uint64_t)p * ws.bsize_stride;
    if (t.n_own > 0) t.x = load_key4(sc, bz, t.i0);
    else { t.x.k[0] = t.x.k[1] = t.x.k[2] = t.x.k[3] = 0u; t.x.z = 0u; }
    return c * TKM_CHUNK < t.nb;                             // the chunk holds blocks of the pair
}

// the state after pick `pass - 1` (pass >= 1) from the state before it and the
// histogram of that pass; the initial state for pass 0.  hl, hd: 2048 words
// of LDS each.
__device__ __forceinline__ TkmHdr tkm_state(const TkmCtx &t, int pass, uint32_t *hl, uint32_t *hd, uint32_t *sbuf) {
    TkmHdr h;
    if (pass == 0) {
        h.base = 0u; h.span = 0xffffffffu; h.rem = (uint32_t)max(t.budget, 0); h.done = t.budget <= 0;
        return h;
    }
    h = ((const TkmHdr *)(t.st + 3 * TOPK_BINS))[pass - 1];
    if (h.done) return h;
    for (int i = threadIdx.x; i < TOPK_BINS; i += 1024) hl[i] = t.st[(pass - 1) * TOPK_BINS + i];
    lds_barrier();
    const int bits = 32 - (h.span ? __builtin_clz(h.span) : 32);
    const int sh = bits > 11 ? bits - 11 : 0;
    h.done = radix_pick(hl, hd, sbuf, sh, h.base, h.span, h.rem) ? 1u : 0u;
    return h;
}

// grid (chunks, pairs): pass 0, 1 or 2 of the radix selection
__global__ void __launch_bounds__(1024) k_tkm_pass(Geom g, WsGeom ws, int pass) {
    __shared__ uint32_t hl[TOPK_BINS], hd[TOPK_BINS], sbuf[64];
    const int p = blockIdx.y, c = blockIdx.x, tid = threadIdx.x;
    TkmCtx t;
    const bool mine = tkm_setup(g, ws, p, c, t);
    if (!mine && c != 0) return;                            // past the pair's blocks (workgroup 0 records the state)
    const TkmHdr h = tkm_state(t, pass, hl, hd, sbuf);
    if (c == 0 && tid == 0) ((TkmHdr *)(t.st + 3 * TOPK_BINS))[pass] = h;
    if (h.done || !mine) return;
    const int bits = 32 - (h.span ? __builtin_clz(h.span) : 32);
    const int sh = bits > 11 ? bits - 11 : 0;
    lds_barrier();                                          // hl (the previous pick's bins) is reused
    for (int i = tid; i < TOPK_BINS; i += 1024) hl[i] = 0u;
    lds_barrier();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t key = t.x.k[e], d = key - h.base;
        if (t.in(e) && key >= h.base && d <= h.span) atomicAdd(&hl[d >> sh], t.x.tok(e));
    }
    lds_barrier();
    uint32_t *hg = t.st + pass * TOPK_BINS;
    for (int i = tid; i < TOPK_BINS; i += 1024)
        if (hl[i]) atomicAdd(&hg[i], hl[i]);
}

// tokens equal to T among the chunk's blocks, in block order: v (this
// thread's four blocks), then the exclusive prefix over the workgroup
__device__ __forceinline__ uint32_t tkm_eq4(const TkmCtx &t, uint32_t T) {
    uint32_t v = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) v += (t.in(e) && t.x.k[e] == T) ? t.x.tok(e) : 0u;
    return v;
}

// grid (chunks, pairs): the last pick (T = base, need = rem), then the tokens
// equal to T per chunk
__global__ void __launch_bounds__(1024) k_tkm_eq(Geom g, WsGeom ws, int nch) {
    __shared__ uint32_t hl[TOPK_BINS], hd[TOPK_BINS], sbuf[64];
    const int p = blockIdx.y, c = blockIdx.x, tid = threadIdx.x;
    TkmCtx t;
    const bool mine = tkm_setup(g, ws, p, c, t);
    if (!mine && c != 0) return;
    const TkmHdr h = tkm_state(t, 3, hl, hd, sbuf);
    if (c == 0 && tid == 0) ((TkmHdr *)(t.st + 3 * TOPK_BINS))[3] = h;
    if (!mine) return;
    uint32_t v[1] = {t.budget > 0 ? tkm_eq4(t, h.base) : 0u}, tot[1];
    block_excl_scan_1024<1>(v, tot, sbuf);
    if (tid == 0) t.st[3 * TOPK_BINS + 16 + c] = tot[0];
}

// sum of the first n counts at x, a lane each (one after the other they were
// most of the list kernel's 14.7 us at 32 chunks)
__device__ __forceinline__ uint32_t sum_first(const uint32_t *x, int n) {
    const int lane = threadIdx.x & 63;
    uint32_t s = 0u;
    for (int i = 0; i < n; i += 64) s += i + lane < n ? x[i + lane] : 0u;
    return (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(s), 63);
}

// the taken mask (bit e: block i0 + e) of this thread's blocks
__device__ __forceinline__ uint32_t tkm_taken(const TkmCtx &t, const TkmHdr &h, int c, uint32_t *sbuf) {
    const uint32_t *eq = t.st + 3 * TOPK_BINS + 16;
    const uint32_t before = sum_first(eq, c);               // equal tokens of the chunks before
    const uint32_t T = h.base, need = h.rem;
    uint32_t v[1] = {t.budget > 0 ? tkm_eq4(t, T) : 0u}, tot[1];
    block_excl_scan_1024<1>(v, tot, sbuf);
    uint32_t acc = before + v[0], m = 0u;
    if (t.budget > 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t key = t.x.k[e];
            const bool eqk = t.in(e) && key == T;
            const bool tk = t.in(e) && (key > T || (eqk && acc < need));
            acc += eqk ? t.x.tok(e) : 0u;
            m |= tk ? (1u << e) : 0u;
        }
    }
    return m;
}

// grid (chunks, pairs): each chunk's taken blocks
__global__ void __launch_bounds__(1024) k_tkm_taken(Geom g, WsGeom ws, int nch) {
    __shared__ uint32_t sbuf[64];
    const int p = blockIdx.y, c = blockIdx.x, tid = threadIdx.x;
    TkmCtx t;
    if (!tkm_setup(g, ws, p, c, t)) return;
    const TkmHdr h = ((const TkmHdr *)(t.st + 3 * TOPK_BINS))[3];
    const uint32_t m = tkm_taken(t, h, c, sbuf);
    uint32_t v[1] = {(uint32_t)__popc(m)}, tot[1];
    block_excl_scan_1024<1>(v, tot, sbuf);
    if (tid == 0) t.st[3 * TOPK_BINS + 16 + nch + c] = tot[0];
}

// grid (chunks, pairs): the list entries of each chunk in block order, their
// record info, and the list position where each window starts
__global__ void __launch_bounds__(1024) k_tkm_write(Geom g, WsGeom ws, int nch) {
    __shared__ uint32_t sbuf[64], tpos[1024], tmk[1024];
    __shared__ int fbw[TOPK_MAXW];
    const int p = blockIdx.y, c = blockIdx.x, tid = threadIdx.x;
    TkmCtx t;
    const bool mine = tkm_setup(g, ws, p, c, t);
    // the record info of this thread's four blocks, loaded with the keys
    // (taken or not): it is not waited on until the list is written
    const uint2 *bi = ws.binfo + (uint64_t)p * (ws.binfo_stride / 8);
    uint2 br[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) br[e] = t.in(e) ? bi[t.i0 + e] : make_uint2(0u, 0u);
    const int nvalid = (t.nb + TKM_CHUNK - 1) / TKM_CHUNK;  // chunks holding blocks
    const uint32_t *tk = t.st + 3 * TOPK_BINS + 16 + nch;
    const uint32_t before = sum_first(tk, min(c, nvalid));
    const uint32_t k = t.budget > 0 ? sum_first(tk, nvalid) : 0u;
    int32_t *wsel = ws.wsel + (uint64_t)p * (ws.wsel_stride / 4);
    const int nwl = min(g.nw, TOPK_MAXW);
    if (c == 0) window_tail(g, t.nb, (int)k, wsel);
    if (!mine && c != 0) return;
    window_firsts<1024>(g, p, t.nb, t.ndesc, nwl, fbw);
    const TkmHdr h = ((const TkmHdr *)(t.st + 3 * TOPK_BINS))[3];
    const uint32_t m = mine ? tkm_taken(t, h, c, sbuf) : 0u;
    uint32_t v[1] = {(uint32_t)__popc(m)}, tot[1];
    block_excl_scan_1024<1>(v, tot, sbuf);                  // (its barriers also publish fbw)
    const uint32_t pos0 = before + v[0];
    int32_t *sel = ws.sel + (uint64_t)p * (ws.sel_stride / 4);
    uint2 *sinfo = ws.selinfo + (uint64_t)p * (ws.selinfo_stride / 8);
    uint32_t pos = pos0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if ((m >> e) & 1u) { sel[pos] = t.i0 + e; sinfo[pos] = br[e]; }
        pos += (m >> e) & 1u;
    }
    tpos[tid] = pos0;
    tmk[tid] = m;
    lds_barrier();
    const int lo = c * TKM_CHUNK, hi = min(lo + TKM_CHUNK, t.nb);
    for (int w = tid; w < nwl; w += 1024) {
        const int f = fbw[w];
        if (f >= lo && f < hi) {
            const int o = f - lo, th = o >> 2, e0 = o & 3;
            wsel[w] = (int)(tpos[th] + (uint32_t)__popc(tmk[th] & ((1u << e0) - 1u)));
        } else if (c == 0 && (f >= t.nb || t.budget <= 0)) {
            wsel[w] = (int)k;
        }
    }
}

// ------------------------------------------------------------------ combine
// Two kernels.  k_combine: one workgroup per (pair p, block of 16 output
// columns j0.., window slot w), 256 threads; slot w = windows is the update
// buffer's split.  It merges the window's splits' (max, sum, accumulator) by
// log-sum-exp, rotates the merged accumulator back once with the window's R_v
// for its columns (x_j = sum_c a_c R_v[c][j]: rows j0.. of the stored R_v^T,
// 8 KB; the rotation stays merged into one vector per window, Sec. 5.3) and
// stores the window's (max, sum, columns) per head.  k_merge then merges the
// windows' results of each output by log-sum-exp.  Kernel boundaries make the
// attention's partials and the window results visible.  Blocks are ordered
// so that b % 8, the XCD a block runs on, is p % 8, as in the attention.
constexpr int CMB_THREADS = 256;

// maximum over the wave on the lane shifts (lanes without a source keep theirs)
__device__ __forceinline__ float wave_max_dpp(float x) {
    auto step = [&](auto c, auto rows) {
        const float o = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(x), __float_as_int(x), decltype(c)::value,
                                                                   decltype(rows)::value, 0xf, false));
        x = fmaxf(x, o);
    };
    step(IntC<0x111>{}, IntC<0xf>{});
    step(IntC<0x112>{}, IntC<0xf>{});
    step(IntC<0x114>{}, IntC<0xf>{});
    step(IntC<0x118>{}, IntC<0xf>{});
    step(IntC<0x142>{}, IntC<0xa>{});
    step(IntC<0x143>{}, IntC<0xc>{});
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}

// one slot's (max, sum, column) into the running merge
__device__ __forceinline__ void merge_slot(float wm, float wl, float y, float &M, float &Lsum, float &o) {
    if (wm == -INFINITY) return;
    const float mn = fmaxf(M, wm);
    const float a = __expf(M - mn), b = __expf(wm - mn);    // M = -inf: a = 0
    o = o * a + y * b;
    Lsum = Lsum * a + wl * b;
    M = mn;
}

//
// NS > 1 (caches of NS - 1 <= 2 windows): one workgroup takes all NS slots of
// its (pair, columns), 256 threads each, and merges them itself, so that the
// second kernel and its launch fall away: 8 x 131072 tokens (two windows) 8.7 +
// 4.8 us apart, 7.5 us fused; with more windows a workgroup per slot spreads
// them over the chip.  The splits of a round get their weights at once, a lane
// each; running maxima in 16-split steps took 26 us where this takes 14 (16
// ragged sequences, groups of 7, fused).
template <int GP, int NS>
__global__ void __launch_bounds__(CMB_THREADS * NS) k_combine(Geom g, WsGeom ws, float *out) {
    constexpr int PS = GP * (D + 2);
    constexpr int NPART = CMB_THREADS / (GP * CMB_COLS);     // threads per output in the rotation
    constexpr int CPP = D / NPART;                            // channels per thread
    constexpr int NE = GP * D / CMB_THREADS;                  // merged elements per thread
    constexpr int CH = 8;                                     // splits whose accumulators are loaded together
    constexpr int CR = 64;                                    // splits of a round: one lane each for their weights
    constexpr int HPW = GP / 4;                               // heads per wave
    static_assert(CMB_THREADS == 256 && GP % 4 == 0, "four waves share the heads");
    static_assert(CMB_COLS * D / 4 == 2 * CMB_THREADS, "two 16-byte pieces of R_v^T rows per thread");
    __shared__ float am_s[NS][GP][D];                         // merged accumulator of the window
    __shared__ float rv_s[NS][CMB_COLS][D + 4];               // R_v[c][j0 + jj] as rows jj
    __shared__ float sm_s[NS][CR][GP + 1], sl_s[NS][CR][GP + 1]; // staged split maxima (then weights) and sums
    __shared__ float wml_s[NS][2][GP], wsc_s[NS][GP];         // the window's running max, sum, rescale
    __shared__ float fin[NS][GP][CMB_COLS];                   // the slots' columns (NS > 1)
    const int np8 = (g.npairs + 7) / 8 * 8;
    const int grp = NS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / CMB_THREADS) : 0;
    const int bid = blockIdx.x, p = bid % np8, cc = (bid / np8) % CMB_NCC, w = NS > 1 ? grp : bid / (np8 * CMB_NCC);
    if (p >= g.npairs) return;
    const int j0 = cc * CMB_COLS, tid = threadIdx.x - grp * CMB_THREADS;
    auto &am = am_s[grp];
    auto &rv = rv_s[grp];
    auto &sm = sm_s[grp];
    auto &sl = sl_s[grp];
    auto &wml = wml_s[grp];
    auto &wsc = wsc_s[grp];
    const int oi = tid / NPART, part_i = tid % NPART;         // output (head, column) and channel part
    const int oh = oi / CMB_COLS, oj = oi % CMB_COLS;
    // R_v[c][j0 .. j0 + 15], loaded before it is known whether the slot has
    // splits, unless its window holds no token (a cache of 64 windows that holds
    // 32 x 1000 tokens would read 512 MB of rotations for nothing)
    const PairMeta meta = *g.meta_of(p);
    const bool turn = w < g.nw && g.rotated && (NS > 1 || (g.dyn ? w < meta.nwin : (long long)w * g.W < meta.L));
    float4 rq0 = make_float4(0.0f, 0.0f, 0.0f, 0.0f), rq1 = rq0;
    if (turn) {
        const float4 *rvt = (const float4 *)(g.rot_of(p, w) + D * D + (uint64_t)j0 * D);
        rq0 = rvt[tid];
        rq1 = rvt[tid + CMB_THREADS];
    }
    int nf, prov, nbuf;
    pair_ndesc(meta, nf, prov, nbuf);
    const int32_t *wsel = ws.wsel + (uint64_t)p * (ws.wsel_stride / 4);
    const float *part = ws.part + (uint64_t)p * (ws.part_stride / 4);
    const int lim = ws.max_blocks;
    float *res = ws.wres + (uint64_t)p * (ws.wres_stride / 4) + ((uint64_t)cc * (g.nw + 1) + w) * (GP * CMB_RES);
    // this slot's splits: the windows' splits are numbered window by window,
    // then the buffer's (the attention's numbering), s0 = those before it
    int s0 = 0, nsp = 0, most = 0;                            // most: splits of the largest slot (the rounds they share)
    // the attention's plan (blocks per split, or one window's fixed splits)
    const int bps = NS == 2 && ws.fix_splits ? 1 : min(max(ws.wsel[g.nw + 2], SPLIT_LEAST), SPLIT_MAX);
    if (NS == 1 && g.nw > 2) {                                // a lane per window (one after the other, most of an empty slot's time)
        const int lane = tid & 63, last = min(w, g.nw - 1);
        for (int x0 = 0; x0 <= last; x0 += 64) {
            const int x = x0 + lane, a = x <= last ? min(max(wsel[x], 0), lim) : 0, b = x <= last ? min(max(wsel[x + 1], a), lim) : 0;
            const uint32_t n = (uint32_t)((b - a + bps - 1) / bps);
            s0 += (int)__builtin_amdgcn_readlane((int)wave_scan_add(x < w ? n : 0u), 63);
            if (w >= x0 && w < x0 + 64) nsp = (int)__builtin_amdgcn_readlane((int)n, w - x0);
        }
    } else {
        for (int x = 0; x <= (NS > 1 ? g.nw - 1 : min(w, g.nw - 1)); ++x) {
            const int a = min(max(wsel[x], 0), lim), b = min(max(wsel[x + 1], a), lim);
            const int n = NS == 2 && ws.fix_splits ? fixed_splits(g, ws, meta.L, b - a) : (b - a + bps - 1) / bps;
            if (x < w) s0 += n; else if (x == w) nsp = n;
            most = max(most, n);
        }
    }
    if (w == g.nw) nsp = nbuf > 0 ? 1 : 0;
    if (s0 + nsp > ws.max_splits) nsp = 0;                    // (cannot happen: the attention had this many)
    if (NS > 1) { most = max(most, 1); } else most = nsp;
    const bool rot = turn && nsp > 0;
    if (NS > 1 || nsp > 0) {
        float A[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e) A[e] = 0.0f;
        const int lane = tid & 63, wv = tid >> 6;
        float Mo[HPW];                                        // running maximum of this wave's heads
#pragma unroll
        for (int x = 0; x < HPW; ++x) Mo[x] = -INFINITY;
        if (tid < GP) wml[1][tid] = 0.0f;
        for (int c0 = 0; c0 < most; c0 += CR) {
            const int n = max(0, min(CR, nsp - c0));
            const float *pc = part + (uint64_t)(s0 + c0) * PS;
            // the first batch of accumulator elements, then the round's maxima and sums into LDS
            float av[CH][NE];
            auto batch = [&](int j0) {
#pragma unroll
                for (int j = 0; j < CH; ++j)
#pragma unroll
                    for (int e = 0; e < NE; ++e)
                        av[j][e] = j0 + j < n ? pc[(uint64_t)(j0 + j) * PS + 2 * GP + tid + e * CMB_THREADS] : 0.0f;
            };
            batch(0);
            for (int i = tid; i < n * GP; i += CMB_THREADS) {
                const float *ps = pc + (uint64_t)(i / GP) * PS;
                sm[i / GP][i % GP] = ps[i % GP];
                sl[i / GP][i % GP] = ps[GP + i % GP];
            }
            lds_barrier();
            // a lane per split, a wave per head (or two): the new maximum, every split's weight, the sum
#pragma unroll
            for (int x = 0; x < HPW; ++x) {
                const int h = wv * HPW + x;
                const float m = lane < n ? sm[lane][h] : -INFINITY;
                const float Mc = fmaxf(Mo[x], wave_max_dpp(m));
                const float f = m == -INFINITY ? 0.0f : __expf(m - Mc);
                const float ls = tree64(lane < n ? f * sl[lane][h] : 0.0f);
                if (lane < n) sm[lane][h] = f;
                if (lane == 0) {
                    const float sc = Mo[x] == -INFINITY ? 0.0f : __expf(Mo[x] - Mc);
                    wsc[h] = sc;
                    wml[0][h] = Mc;
                    wml[1][h] = wml[1][h] * sc + ls;
                }
                Mo[x] = Mc;
            }
            lds_barrier();
#pragma unroll
            for (int e = 0; e < NE; ++e) A[e] *= wsc[(tid + e * CMB_THREADS) / D];
            for (int j0 = 0; j0 < n; j0 += CH) {
                float cur[CH][NE];
#pragma unroll
                for (int j = 0; j < CH; ++j)
#pragma unroll
                    for (int e = 0; e < NE; ++e) cur[j][e] = av[j][e];
                if (j0 + CH < n) batch(j0 + CH);
#pragma unroll
                for (int j = 0; j < CH; ++j)
                    if (j0 + j < n) {
#pragma unroll
                        for (int e = 0; e < NE; ++e) A[e] = fmaf(cur[j][e], sm[j0 + j][(tid + e * CMB_THREADS) / D], A[e]);
                    }
            }
            if (c0 + CR < most) lds_barrier();                // sm, sl, wsc are rewritten next
        }
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            const int i = tid + e * CMB_THREADS;
            am[i / D][i % D] = A[e];
        }
        if (rot) {                                            // (rows of R_v^T: 16 x 32 pieces)
            *(float4 *)&rv[tid / (D / 4)][4 * (tid % (D / 4))] = rq0;
            *(float4 *)&rv[(tid + CMB_THREADS) / (D / 4)][4 * ((tid + CMB_THREADS) % (D / 4))] = rq1;
        }
        lds_barrier();
        float y = 0.0f;
        if (rot) {
#pragma unroll 8
            for (int c = part_i * CPP; c < (part_i + 1) * CPP; ++c) y = fmaf(am[oh][c], rv[oj][c], y);
#pragma unroll
            for (int m = 1; m < NPART; m <<= 1) y += __shfl_xor(y, m, WAVE);
        } else {
            y = am[oh][j0 + oj];
        }
        if (NS > 1) {
            if (part_i == 0) fin[grp][oh][oj] = y;
            lds_barrier();
            if (grp == 0 && part_i == 0 && oh < g.G) {        // the slots in order, as the merge kernel takes them
                float M = -INFINITY, Lsum = 0.0f, o = 0.0f;
#pragma unroll
                for (int x = 0; x < NS; ++x) merge_slot(wml_s[x][0][oh], wml_s[x][1][oh], fin[x][oh][oj], M, Lsum, o);
                out[((uint64_t)p * g.G + oh) * D + j0 + oj] = (Lsum > 0.0f) ? o / Lsum : 0.0f;
            }
            return;
        }
        if (part_i == 0) res[oh * CMB_RES + 2 + oj] = y;
        if (tid < GP) { res[tid * CMB_RES] = wml[0][tid]; res[tid * CMB_RES + 1] = wml[1][tid]; }
    } else if (tid < GP) {                                    // an empty slot
        res[tid * CMB_RES] = -INFINITY;
        res[tid * CMB_RES + 1] = 0.0f;
    }
}

// one thread per output (pair, head, column): the log-sum-exp merge of its
// window slots' results, in slot order; the slots are read twenty per round
// trip (a long context has dozens of windows)
template <int GP>
__global__ void __launch_bounds__(256) k_merge(Geom g, WsGeom ws, float *out) {
    constexpr int MU = 20;                                    // (a million tokens: 17 slots, one round trip)
    const int i = blockIdx.x * 256 + threadIdx.x;
    const int p = i / (GP * D), h = (i / D) % GP, j = i % D;
    if (p >= g.npairs || h >= g.G) return;
    const int cc = j / CMB_COLS, jj = j % CMB_COLS;
    const float *r = ws.wres + (uint64_t)p * (ws.wres_stride / 4) + (uint64_t)cc * (g.nw + 1) * (GP * CMB_RES)
                     + h * CMB_RES;
    float M = -INFINITY, Lsum = 0.0f, o = 0.0f;
    for (int x0 = 0; x0 <= g.nw; x0 += MU) {
        float wm[MU], wl[MU], y[MU];
#pragma unroll
        for (int u = 0; u < MU; ++u) {
            wm[u] = -INFINITY; wl[u] = 0.0f; y[u] = 0.0f;
            if (x0 + u <= g.nw) {
                const float *rr = r + (uint64_t)(x0 + u) * (GP * CMB_RES);
                wm[u] = rr[0]; wl[u] = rr[1]; y[u] = rr[2 + jj];
            }
        }
#pragma unroll
        for (int u = 0; u < MU; ++u) {
            merge_slot(wm[u], wl[u], y[u], M, Lsum, o);
        }
    }
    out[((uint64_t)p * g.G + h) * D + j] = (Lsum > 0.0f) ? o / Lsum : 0.0f;
}

int max_keep(const Geom &g) {
    int r = g.def_keep;
    for (int i = 0; i < 3; ++i) r = max(r, g.keep_cand[i]);
    return r;
}

// attention workgroups the device holds at once: ATTN_WPE waves per SIMD,
// four SIMDs per compute unit, ATTN_NWV waves per workgroup
int attn_slots() {
    static int cached[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) dev = 0;
    const int d = dev & 63;
    if (cached[d] == 0) {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
        cached[d] = cus * 4 * ATTN_WPE / ATTN_NWV;
    }
    return cached[d];
}

template <int GP>
hipError_t launch_decode_gp(const Geom &g, const WsGeom &w_in, const uint16_t *q, float *out, float scale,
                            int max_desc_used, int max_windows_used, hipStream_t s, hipEvent_t *ev) {
    WsGeom w = w_in;
    w.split_slots = attn_slots();
    w.fix_splits = 0;
    const int nwq = g.rotated ? max_windows_used : 1;
    const bool small = max_keep(g) <= 48;
    bool fixed = true;                         // every possible kept count in {16, 32, 48}
    for (int i = 0; i < 4; ++i) {
        const int r = i < 3 ? g.keep_cand[i] : g.def_keep;
        fixed = fixed && (r == 16 || r == 32 || r == 48);
    }
    if (ev) (void)hipEventRecord(ev[0], s);
    // blocks of a pair at most in this call: its segments times the most
    // blocks a segment can have
    int minb = g.def_block;
    for (int i = 0; i < 3; ++i) minb = min(minb, g.block_cand[i]);
    const long long maxb = (long long)max_desc_used * (SEG / minb);
    // One window per pair: splits of about the same tokens for every pair, at
    // least 128 of them and as many as fill the chip once, planned here.  The
    // attention's workgroups then read their own pair's counts only instead of
    // deriving the call's plan from all pairs': 1 x 4117 tokens 18.4 -> 13.0 us
    // (with the finer splits), 8 requests of 1000 tokens 11.3 -> 9.7.  Batches so ragged that most places would
    // stay empty keep the derived plan.
    if (g.nw == 1 && max_desc_used > 0) {
        const long long avail = std::max(w.split_slots - g.npairs, std::max(w.split_slots / 4, 1));
        const long long tok = std::max<long long>(128, (g.sel_tokens + avail - 1) / avail);
        const long long n = (long long)max_desc_used * SEG, longest = std::min(n, n * g.sel_num / g.sel_den + 1);
        const long long most = std::max((longest + tok - 1) / tok + 1, (longest / minb + SPLIT_MAX) / SPLIT_MAX + 1);
        const long long fix = std::min<long long>(most, w.max_splits - 1);
        if (g.npairs * (fix + 1) <= 4ll * w.split_slots) {
            w.fix_splits = (int)fix;
            w.split_tok = (float)tok;
        }
    }
    hipError_t e = hipSuccess;
    const int cus = w.split_slots * ATTN_NWV / (4 * ATTN_WPE);
    if (fixed && g.nw == 1 && maxb <= FRONT_BLOCKS && g.npairs <= cus) {
        // a short context: rotation, scores and selection of a pair by one
        // workgroup (timed as the scoring), as long as every pair has a compute
        // unit to itself.  us a step with this kernel and with the three:
        //   sequences of 8 kv heads    1 x 1000  1 x 8100  32 x 1000  32 x 8100
        //     this                       28.4      39.3       40.6       64.2
        //     the three                  32.2      40.8       46.4       73.8
        //                             40 x 1000  40 x 8100  64 x 1000  128 x 1000
        //     this                       56.8      83.9       66.1      119.9
        //     the three                  52.1      90.6       62.6       98.4
        // (2048 blocks are what its LDS holds.  The host counts a pair's blocks as
        // its segments' smallest candidates, so a call may have far fewer.)
        if (ev) (void)hipEventRecord(ev[1], s);
        if ((e = launch_front(g, w, q, s)) != hipSuccess) return e;
        if (ev) (void)hipEventRecord(ev[2], s);
    } else {
        hipLaunchKernelGGL(k_qrot, dim3(nwq * (D / QROT_COLS), g.npairs), dim3(256), 0, s, g, w, q);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (ev) (void)hipEventRecord(ev[1], s);
        if (max_desc_used > 0 && (e = launch_score(g, w, max_desc_used, fixed, small, s)) != hipSuccess) return e;
        if (ev) (void)hipEventRecord(ev[2], s);
        if (maxb > 1024 * TOPK_KPT_MAX) {
            if (!w.tkx) return hipErrorInvalidValue;               // the workspace has no multi-workgroup state
            const int nch = ceil_div(w.max_blocks, TKM_CHUNK);
            const dim3 grid(nch, g.npairs);
            for (int pass = 0; pass < 3; ++pass) {
                hipLaunchKernelGGL(k_tkm_pass, grid, dim3(1024), 0, s, g, w, pass);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
            hipLaunchKernelGGL(k_tkm_eq, grid, dim3(1024), 0, s, g, w, nch);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL(k_tkm_taken, grid, dim3(1024), 0, s, g, w, nch);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL(k_tkm_write, grid, dim3(1024), 0, s, g, w, nch);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        } else {
            hipLaunchKernelGGL(k_topk, dim3(g.npairs), dim3(1024), 0, s, g, w);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    if (ev) (void)hipEventRecord(ev[3], s);
    if (g.dtype) e = GP == 4 ? launch_attn_bf16_g4(g, w, scale, q, fixed, small, s) : launch_attn_bf16_g8(g, w, scale, q, fixed, small, s);
    else e = GP == 4 ? launch_attn_fp16_g4(g, w, scale, q, fixed, small, s) : launch_attn_fp16_g8(g, w, scale, q, fixed, small, s);
    if (e != hipSuccess) return e;
    if (ev) (void)hipEventRecord(ev[4], s);
    // Few slots per output: one kernel.  Three slots of eight heads are 12 waves of
    // 118 registers, one workgroup per compute unit: that form is for two rounds
    // of them at most.  us of the merge fused / apart, groups of 8, two windows:
    //   pairs   8          64           128          264          560
    //         9.0 / 11.6  14.1 / 16.2  23.6 / 22.1  47.1 / 36.1  89.8 / 63.5
    const int wgs = (g.npairs + 7) / 8 * 8 * CMB_NCC;
    if (g.nw == 1 || (g.nw == 2 && (GP == 4 || wgs <= 2 * cus))) {
        if (g.nw == 1) hipLaunchKernelGGL((k_combine<GP, 2>), dim3(wgs), dim3(2 * CMB_THREADS), 0, s, g, w, out);
        else hipLaunchKernelGGL((k_combine<GP, 3>), dim3(wgs), dim3(3 * CMB_THREADS), 0, s, g, w, out);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    } else {
        hipLaunchKernelGGL((k_combine<GP, 1>), dim3(wgs * (g.nw + 1)), dim3(CMB_THREADS), 0, s, g, w, out);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(k_merge<GP>, dim3(ceil_div(g.npairs * GP * D, 256)), dim3(256), 0, s, g, w, out);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (ev) (void)hipEventRecord(ev[5], s);
    return hipSuccess;
}

}  // namespace

hipError_t launch_decode(const Geom &g, const WsGeom &w, const uint16_t *q, float *out, float scale,
                         int max_desc_used, int max_windows_used, hipStream_t s, hipEvent_t *ev) {
    if (g.GP == 4) return launch_decode_gp<4>(g, w, q, out, scale, max_desc_used, max_windows_used, s, ev);
    return launch_decode_gp<8>(g, w, q, out, scale, max_desc_used, max_windows_used, s, ev);
}

}  // namespace mosaic
