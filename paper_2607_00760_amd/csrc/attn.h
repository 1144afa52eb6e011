// attn.h -- the decode step's attention over the selected blocks and the
// update buffer (Sec. 5.3); each attn_*.hip instantiates one (dtype, padded
// group) pair (not part of the C ABI).
//
// Split-K over the selected list (up to 128 blocks of one rotation window per
// split).  The split's blocks are ordered by size, so a 64-token chunk never
// cuts a block and a token finds its block by a closed form.  Lane per token:
// the packed K record is expanded from registers into an LDS tile with the
// bitmap walk, logits K . q^T on the matrix cores (16x16x32, q split into two
// 16-bit halves), online softmax in fp32 on the accumulator layout, then V
// expanded the same way and P . V on the matrix cores.  The matrix-core
// operand reads zero what they read, so the tile is zero again for the next
// expansion without a clearing pass.  The next chunk's records are loaded
// while the current one is processed.  The update buffer is one more split
// (dense, unrotated).
#pragma once
#include "decode_common.h"

namespace mosaic {

namespace {

// ------------------------------------------------------------------ attention
// a selected block in the attention kernel's LDS table: byte offset in the
// pair's token arena, and r << 8 | log2g << 16 | log2b << 20
typedef uint2 BlkInfo;

// Split-K plan of a call.  A window of a pair with n selected entries gets
// ceil(n / bps) splits of at most bps blocks, dealt round-robin, so every split of
// a window holds the same mix of 16-, 8- and 4-token blocks (the list is in block
// order, where blocks of one size cluster); a pair's splits are its windows' in
// order, then one for its update buffer.  Three plans, one numbering:
//   fixed     (caches of one window, unless very uneven; planned by the host,
//             fixed_splits): each pair's tokens in shares of the same size, at
//             least 128, of at most SPLIT_MAX blocks; a workgroup needs its own
//             pair's counts only;
//   register  (up to 128 pairs of up to 16 windows, plan_small): one bps for the
//             call, such that the splits fill whole rounds of the workgroups that
//             the device runs at once (split_slots, less a rounding split for
//             every non-empty window and buffer), from about 128 tokens to
//             SPLIT_MAX blocks;
//   general   (beyond, split_blocks): one bps for the call, one round, within
//             [SPLIT_MIN, SPLIT_MAX].
// The combine takes the fixed plan's numbers from the same function, the others'
// bps from pair 0's list header.  List bounds are clamped to [0, lim] (the list's
// capacity), so that no workspace content can send an index outside it.

// f(n) for the selected entries n of each window of a pair, in window order
// (eight windows' bounds per round trip)
template <typename F>
__device__ __forceinline__ void for_windows(const int32_t *wsel, int nw, int lim, F f) {
    for (int w0 = 0; w0 < nw; w0 += 8) {
        int v[9];
#pragma unroll
        for (int i = 0; i <= 8; ++i) v[i] = wsel[min(w0 + i, nw)];
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (w0 + i < nw) {
                const int a = min(max(v[i], 0), lim), b = min(max(v[i + 1], a), lim);
                f(b - a);
            }
    }
}

// block-wide sum over blockDim.x threads (a multiple of 64); red: 16 words of LDS
__device__ __forceinline__ int block_sum(int v, int *red) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nwv = blockDim.x >> 6;
    const int x = (int)__builtin_amdgcn_readlane((int)wave_scan_add((uint32_t)v), 63);
    if (lane == 0) red[wv] = x;
    __syncthreads();
    int t = 0;
    for (int i = 0; i < nwv; ++i) t += red[i];
    __syncthreads();
    return t;
}

__device__ __forceinline__ bool pair_has_buf(const Geom &g, int p) {
    int nf, prov, nbuf;
    pair_ndesc(*g.meta_of(p), nf, prov, nbuf);
    return nbuf > 0;
}

__device__ __forceinline__ const int32_t *wsel_of(const WsGeom &ws, int p) { return ws.wsel + (uint64_t)p * (ws.wsel_stride / 4); }

// blocks per split of this call (every thread of the block gets it)
__device__ __forceinline__ int split_blocks(const Geom &g, const WsGeom &ws, int *red) {
    int ksum = 0, extra = 0;
    for (int p = threadIdx.x; p < g.npairs; p += blockDim.x) {
        const bool buf = pair_has_buf(g, p);
        for_windows(wsel_of(ws, p), g.nw, ws.max_blocks, [&](int n) { ksum += n; extra += n > 0 ? 1 : 0; });
        extra += buf ? 1 : 0;
    }
    ksum = block_sum(ksum, red);
    extra = block_sum(extra, red);
    const int avail = max(ws.split_slots - extra, max(ws.split_slots / 4, 1));
    return min(max((ksum + avail - 1) / avail, SPLIT_MIN), SPLIT_MAX);
}

// splits of pair p's windows (nbuf > 0 adds the buffer's)
__device__ __forceinline__ int pair_splits(const Geom &g, const WsGeom &ws, int p, int bps) {
    const bool buf = pair_has_buf(g, p);
    int t = 0;
    for_windows(wsel_of(ws, p), g.nw, ws.max_blocks, [&](int n) { t += (n + bps - 1) / bps; });
    return t + (buf ? 1 : 0);
}

// workgroup gidx of the flattened plan -> its pair and the split's index in
// the pair, or p = -1 past the last split; scan: 16 words of LDS
__device__ __forceinline__ void plan_locate(const Geom &g, const WsGeom &ws, int bps, int gidx, int *scan,
                                            int &p_out, int &s_out) {
    __shared__ int loc[2];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nwv = blockDim.x >> 6;
    if (tid == 0) { loc[0] = -1; loc[1] = 0; }
    int carry = 0;
    for (int p0 = 0; p0 < g.npairs; p0 += blockDim.x) {     // block order: uniform trip count
        const int p = p0 + tid;
        const int n = p < g.npairs ? pair_splits(g, ws, p, bps) : 0;
        const uint32_t x = wave_scan_add((uint32_t)n);
        if (lane == 63) scan[wv] = (int)x;
        __syncthreads();
        int before = carry, tot = 0;
        for (int i = 0; i < nwv; ++i) { before += i < wv ? scan[i] : 0; tot += scan[i]; }
        const int first = before + (int)x - n;                 // this pair's first workgroup
        if (n > 0 && gidx >= first && gidx < first + n) { loc[0] = p; loc[1] = gidx - first; }
        carry += tot;
        __syncthreads();
    }
    p_out = loc[0];
    s_out = loc[1];
}

// split s of pair p: window w and its entries e0, e0 + stride, e0 + 2 stride,
// ... (cnt of them); w = -2 past the windows' splits (total of them)
__device__ __forceinline__ void split_of(const int32_t *wsel, int nw, int s, int lim, int bps, int &w_out, int &e0,
                                         int &stride, int &cnt, int &total) {
    int acc = 0;
    w_out = -2; e0 = 0; stride = 1; cnt = 0;
    for (int w = 0; w < nw; ++w) {
        const int a = min(max(wsel[w], 0), lim), b = min(max(wsel[w + 1], a), lim);
        const int nsp = (b - a + bps - 1) / bps;
        if (w_out == -2 && s < acc + nsp) {
            const int k = s - acc;
            w_out = w;
            e0 = a + k;
            stride = nsp;
            cnt = (b - a - k + nsp - 1) / nsp;
        }
        acc += nsp;
    }
    total = acc;
}

// What an attention workgroup does: split s of pair p -- cnt entries e0, e0 +
// stride, ... of window w's list (w = -2: the update buffer when buf is set,
// nothing otherwise) -- or p = -1 past the plan.
struct SplitJob {
    int p, s, w, e0, stride, cnt, L, buf;
};
constexpr int PLAN_W = 16;               // windows whose bounds a thread holds in registers
__host__ __device__ __forceinline__ bool register_plan(const Geom &g) { return g.npairs <= 64 * ATTN_NWV && g.nw <= PLAN_W; }

// The plan and this workgroup's place in it, for at most blockDim.x pairs of
// at most PLAN_W windows: thread p loads pair p's length and window bounds
// once (one round trip; the general functions above read them three times), every division is a multiplication, and the
// thread that finds the workgroup's split publishes it.  Unlike the general
// plan's splits of at least SPLIT_MIN blocks these go down to about 128
// tokens, so short selections use the whole chip: 4 x 32768 tokens with every
// channel kept, 160 workgroups of 768 tokens, 81 us, then 410 of 128, 24 us
// (with the rows taken as the dense kernel takes them).  red: 16 words of LDS.
__device__ __forceinline__ int plan_small(const Geom &g, const WsGeom &ws, int gidx, int *red, SplitJob *job) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, nwv = blockDim.x >> 6, lim = ws.max_blocks;
    const bool on = tid < g.npairs;
    int n[PLAN_W + 1], a0 = 0, L = 0;
    if (on) {
        const int32_t *wsel = wsel_of(ws, tid);
        L = g.meta_of(tid)->L;
#pragma unroll
        for (int i = 0; i <= PLAN_W; ++i) n[i] = wsel[min(i, g.nw)];
        a0 = n[0];
    } else {
#pragma unroll
        for (int i = 0; i <= PLAN_W; ++i) n[i] = 0;
    }
    const int rem = L % SEG, nbuf = rem - (rem >= UBUF ? UBUF : 0);
    int ksum = 0, extra = nbuf > 0 ? 1 : 0;
    a0 = min(max(a0, 0), lim);
    {
        int lo = a0;
#pragma unroll
        for (int i = 0; i < PLAN_W; ++i) {                     // n[i]: entries of window i
            const int hi = min(max(n[i + 1], lo), lim);
            n[i] = hi - lo;
            lo = hi;
            ksum += n[i];
            extra += n[i] > 0 ? 1 : 0;
        }
    }
    const uint32_t ks = wave_scan_add((uint32_t)ksum), ex = wave_scan_add((uint32_t)extra);
    const uint32_t sg = wave_scan_add((uint32_t)(L / UBUF)), nm = wave_max_u((uint32_t)ksum);
    if (tid == 0) job->p = -1;
    if (lane == 63) { red[wv] = (int)ks; red[2 + wv] = (int)ex; red[4 + wv] = (int)sg; red[6 + wv] = (int)nm; }
    lds_barrier();
    int kt = 0, et = 0, st = 0, nmax = 0;
    for (int i = 0; i < nwv; ++i) { kt += red[i]; et += red[2 + i]; st += red[4 + i]; nmax = max(nmax, red[6 + i]); }
    const int avail = max(ws.split_slots - et, max(ws.split_slots / 4, 1));
    // no split below about 128 tokens (a chunk for each of its waves) at the
    // blocks' mean size, nor so small that a pair's splits outgrow its array,
    // which is sized for split_min blocks of the smallest size
    const float tokens = (float)st * UBUF * g.sel_num / g.sel_den;
    const int b128 = (int)(128.0f * (float)kt / fmaxf(tokens, 1.0f) + 0.5f);
    const int fit = (int)(((long long)nmax * ws.split_min + ws.max_sel - 1) / ws.max_sel);
    // more than SPLIT_MAX blocks for each resident workgroup: as many whole
    // rounds as that takes, of equal splits (a last round of a few splits
    // costs as much as a full one: a million tokens, 1037 splits of 128 blocks
    // for 1024 workgroups, 84 us; two rounds of 60 blocks, 72 us)
    const int rounds = (kt + avail * SPLIT_MAX - 1) / (avail * SPLIT_MAX);
    const int room = rounds > 1 ? rounds * ws.split_slots - min(et, ws.split_slots) : avail;
    const int bps = min(max(max((kt + room - 1) / room, fit), min(max(b128, SPLIT_LEAST), SPLIT_MIN)), SPLIT_MAX);
    const uint32_t inv = 0xffffffffu / (uint32_t)bps + 1u;      // x / bps = umulhi(x, inv) for x * bps < 2^32
    auto splits = [&](int c) { return (int)__umulhi((uint32_t)(c + bps - 1), inv); };
    int ns = nbuf > 0 ? 1 : 0;
#pragma unroll
    for (int i = 0; i < PLAN_W; ++i) ns += splits(n[i]);
    const uint32_t x = wave_scan_add((uint32_t)ns);
    if (lane == 63) red[8 + wv] = (int)x;
    lds_barrier();
    int first = (int)x - ns;
    for (int i = 0; i < nwv; ++i) first += i < wv ? red[8 + i] : 0;
    if (gidx >= first && gidx < first + ns) {
        const int s = gidx - first;
        SplitJob j = {tid, s, -2, 0, 1, 0, L, nbuf > 0 ? 1 : 0};
        int acc = 0, a = a0;
#pragma unroll
        for (int i = 0; i < PLAN_W; ++i) {
            const int nsp = splits(n[i]), k = s - acc;
            if (k >= 0 && k < nsp) {
                j.w = i; j.e0 = a + k; j.stride = nsp;
                j.cnt = (n[i] - k + nsp - 1) / nsp;
            }
            acc += nsp;
            a += n[i];
        }
        *job = j;
    }
    lds_barrier();
    return bps;
}

constexpr int CH_TOK = 64;           // tokens per chunk (one wave, lane per token)
constexpr int KT_STRIDE = 136;       // u16 per token row of the K tile (128 + 8 pad)
constexpr int VT_STRIDE = 68;        // u16 per channel row of the V tile (64 + 4 pad)
constexpr int TILE_BYTES = 17408;    // max(64 * 272, 128 * 136)
// block table [SPLIT_MAX] + per-wave class counts (16-byte multiple)
constexpr int ATTN_HDR_BYTES = (8 * SPLIT_MAX + ATTN_NWV * 4 * 4 + 15) / 16 * 16;
static_assert(SPLIT_MAX <= 64 * ATTN_NWV, "one setup thread per block of a split");

// x = hi + lo with hi, lo in the MFMA's 16-bit type (round to nearest even);
// hi + lo carries x to ~16 (bf16) or ~22 (fp16) significant bits
template <int DT>
__device__ __forceinline__ void split8(const float (&x)[8], typename Mma<DT>::v8 &hi, typename Mma<DT>::v8 &lo) {
    using M8 = typename Mma<DT>::v8;
    using E = typename Mma<DT>::el;
    M8 h, l;
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = (E)x[i];
#pragma unroll
    for (int i = 0; i < 8; ++i) l[i] = (E)(x[i] - (float)h[i]);
    hi = h;
    lo = l;
}

// Expand a packed vector into an LDS tile at base + off: COL = false puts
// channel c at + 2c (a token-major row of the K tile), COL = true at
// + c * VT_STRIDE * 2 (a column of the channel-major V tile).  RV as in the
// score walk.
template <int RMAX, int L2G, int RV, bool COL>
__device__ __forceinline__ void scatter_walk(const PVec<RMAX> &x, int r, uint32_t addr) {
    constexpr int GS = 1 << L2G, NWD = 4 >> L2G;
    constexpr uint32_t CB = COL ? VT_STRIDE * 2 : 2;           // bytes per channel
    Walk wk = make_walk<NWD>(x.bw, addr, 32u * GS * CB);
    const int n = RV ? RV : r;
#pragma unroll
    for (int k = 0; k < (RV ? RV : RMAX) / GS; ++k) {
        if (RV || k * GS < n) {                               // wave-uniform
            const uint32_t dst = wk.a + wk.pos() * (GS * CB);
            if (!COL && GS == 1) lds_st<uint16_t>(dst, (uint16_t)half_at(x.v, k));
            else if (!COL && GS == 2) lds_st<uint32_t>(dst, x.v[k]);
            else if (!COL) lds_st<u32x2>(dst, u32x2{x.v[2 * k], x.v[2 * k + 1]});
            else {
#pragma unroll
                for (int e = 0; e < GS; ++e) lds_st<uint16_t>(dst + e * CB, (uint16_t)half_at(x.v, k * GS + e));
            }
            wk.template step<NWD>();
            __builtin_amdgcn_sched_barrier(0);       // keep the steps in order: short live ranges
        }
    }
}

template <int RMAX, int L2G, bool COL, bool FR>
__device__ __forceinline__ void scatter_r(const PVec<RMAX> &x, int r, uint32_t addr) {
    if (FR) {
        if (r == 32) scatter_walk<RMAX, L2G, 32, COL>(x, r, addr);
        else if (r == 16) scatter_walk<RMAX, L2G, 16, COL>(x, r, addr);
        else scatter_walk<RMAX, L2G, (RMAX >= 48 ? 48 : 16), COL>(x, r, addr);
    } else {
        scatter_walk<RMAX, L2G, 0, COL>(x, r, addr);
    }
}

// called by the lanes that hold a token; one pass per distinct (r, log2g)
template <int RMAX, bool COL, bool FR>
__device__ __forceinline__ void scatter_any(const PVec<RMAX> &x, int r, int l2g, uint32_t addr) {
    const int key = (r << 2) | l2g;
    uint64_t todo = __ballot(1);
    while (todo) {
        const int kv = __builtin_amdgcn_readlane(key, (int)__builtin_ctzll(todo));
        const bool mine = key == kv;
        todo &= ~__ballot(mine);
        if (mine) {
            const int rv = kv >> 2;
            if ((kv & 3) == 0) scatter_r<RMAX, 0, COL, FR>(x, rv, addr);
            else if ((kv & 3) == 1) scatter_r<RMAX, 1, COL, FR>(x, rv, addr);
            else scatter_r<RMAX, 2, COL, FR>(x, rv, addr);
        }
    }
}

// where this lane's token of a chunk lives: its block's byte offset in the
// pair's token arena and (token in block, r, log2g, log2b) packed in a word
struct TokLoc {
    uint32_t base, info;
    bool valid;
    __device__ __forceinline__ int j() const { return info & 0xff; }
    __device__ __forceinline__ int r() const { return (info >> 8) & 0xff; }
    __device__ __forceinline__ int l2g() const { return (info >> 16) & 0xf; }
    __device__ __forceinline__ int l2b() const { return info >> 20; }
};

// load the packed K (V when V_ is set) vector of a located token
template <int RMAX, int RL>
__device__ __forceinline__ void load_tok(PVec<RMAX> &x, const uint8_t *tokg, const TokLoc &L, bool V_, int rmax, int T) {
    const int r = L.r(), l2g = L.l2g(), B = 1 << L.l2b(), bmb = bm_bytes(l2g, T), j = L.j();
    const uint32_t half = V_ ? (uint32_t)(B * (bmb + 2 * r)) : 0u;
    const uint8_t *b = tokg + L.base + half;
    load_pvec<RMAX, RL ? 1 : 0, false, RL>(x, b + j * bmb, b + B * bmb + j * 2 * r, rmax, false);
}

// the same for a record with E4M3 values: r bytes of values.  RL > 0: the
// first RL / 2 16-byte granules (8 RL codes, as many values as RL granules
// of 16-bit values), at any 4-byte aligned record; else dword loads of every
// word below rmax, the others from the start of the values again.
template <int RMAX, int RL>
__device__ __forceinline__ void load_tok(PVec8<RMAX> &x, const uint8_t *tokg, const TokLoc &L, bool V_, int rmax, int T) {
    static_assert(RL % 2 == 0 && RL <= RMAX / 8, "whole 16-byte granules of codes");
    const int r = L.r(), l2g = L.l2g(), B = 1 << L.l2b(), bmb = bm_bytes(l2g, T), j = L.j();
    const uint8_t *b = tokg + L.base + (V_ ? (uint32_t)(B * (bmb + r)) : 0u);
    const uint8_t *bm = b + j * bmb, *val = b + B * bmb + j * r;
    if constexpr (RL > 0) {
        const u32x4a4 bb = *(const u32x4a4 *)bm;
        x.bw[0] = bb.x; x.bw[1] = bb.y; x.bw[2] = bb.z; x.bw[3] = bb.w;
        const u32x4a4 *v4 = (const u32x4a4 *)val;
#pragma unroll
        for (int k = 0; k < RL / 2; ++k) {
            const u32x4a4 t = v4[k];
            x.v[4 * k] = t.x; x.v[4 * k + 1] = t.y; x.v[4 * k + 2] = t.z; x.v[4 * k + 3] = t.w;
        }
    } else {
        load_dwords_any<4>(bm, x.bw);                    // a truncated bitmap can sit at any byte
        const uint32_t *v = (const uint32_t *)val;       // token values stay 4-byte aligned
#pragma unroll
        for (int k = 0; k < RMAX / 4; ++k) x.v[k] = v[(4 * k < rmax) ? k : 0];
    }
}

// walk a loaded record into the tile (widening E4M3 codes first)
template <int DT, int RMAX, int RL, bool COL, bool FR>
__device__ __forceinline__ void scatter_rec(const PVec<RMAX> &x, int r, int l2g, uint32_t addr) {
    scatter_any<RMAX, COL, FR>(x, r, l2g, addr);
}
template <int DT, int RMAX, int RL, bool COL, bool FR>
__device__ __forceinline__ void scatter_rec(const PVec8<RMAX> &c, int r, int l2g, uint32_t addr) {
    PVec<RMAX> x;
    widen<DT, RMAX, (RL > 0 ? 2 * RL : RMAX / 4)>(c, x);
    scatter_any<RMAX, COL, FR>(x, r, l2g, addr);
}

// RMAX: the largest kept count, or 0 where every block keeps all D channels
template <int DT, int GP, int RMAX, bool FR, bool F8>
__global__ void __launch_bounds__(64 * ATTN_NWV) __attribute__((amdgpu_waves_per_eu(ATTN_WPE)))
k_attn(Geom g, WsGeom ws, float scale, const uint16_t *qraw) {
    using M8 = typename Mma<DT>::v8;
    constexpr int NWV = ATTN_NWV;
    extern __shared__ __align__(16) uint8_t smem[];
    BlkInfo *blk = (BlkInfo *)smem;                         // [SPLIT_MAX], ordered 16, 8, 4
    int *wcnt = (int *)(smem + 8 * SPLIT_MAX);              // [NWV][4] blocks per size class
    uint8_t *wbase = smem + ATTN_HDR_BYTES;                 // [NWV] tiles
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, q4 = lane >> 4;
    uint8_t *tile = wbase + wave * TILE_BYTES;

    // the call's plan: workgroup b takes the b-th split of the flattened list
    // (pairs in order, each pair's splits in order); the grid covers every plan
    __shared__ SplitJob job;
    __shared__ int red[16];
    if (ws.fix_splits) {
        // one window: every pair has fix_splits places and one for its buffer,
        // and a workgroup needs its own pair's counts only.  All pairs' first
        // places come first, then their second ones, so that work is dealt to
        // every XCD.  Pair by pair, with four places a pair, the ones that held
        // work fell on the same two XCDs: 512 pairs of 6000 tokens 91 us here,
        // now 40; 256 pairs of 8100 tokens 42 and 30.
        SplitJob j;
        j.p = blockIdx.x % g.npairs;
        const int i = blockIdx.x / g.npairs;
        const int32_t *wsel = wsel_of(ws, j.p);
        j.L = g.meta_of(j.p)->L;
        const int a = min(max(wsel[0], 0), ws.max_blocks), n = min(max(wsel[1], a), ws.max_blocks) - a;
        const int sp = fixed_splits(g, ws, j.L, n);
        const int rem = j.L % SEG;
        j.buf = i == ws.fix_splits && rem - (rem >= UBUF ? UBUF : 0) > 0;
        if (i == ws.fix_splits ? !j.buf : i >= sp) return;      // (the whole workgroup)
        j.s = j.buf ? sp : i;
        j.w = j.buf ? -2 : 0;
        j.e0 = a + i;
        j.stride = sp;
        j.cnt = j.buf ? 0 : (n - i + sp - 1) / sp;
        if (tid == 0) job = j;
        lds_barrier();
    } else if (register_plan(g)) {
        const int bps = plan_small(g, ws, blockIdx.x, red, &job);
        if (blockIdx.x == 0 && tid == 0) ws.wsel[g.nw + 2] = bps;    // for the combine (pair 0's list header)
    } else {
        const int bps = split_blocks(g, ws, red);
        if (blockIdx.x == 0 && tid == 0) ws.wsel[g.nw + 2] = bps;
        SplitJob j;
        plan_locate(g, ws, bps, blockIdx.x, red, j.p, j.s);
        if (j.p >= 0) {
            int nf, prov, nbuf, total;
            j.L = g.meta_of(j.p)->L;
            pair_ndesc(*g.meta_of(j.p), nf, prov, nbuf);
            split_of(wsel_of(ws, j.p), g.nw, j.s, ws.max_blocks, bps, j.w, j.e0, j.stride, j.cnt, total);
            j.buf = j.w == -2 && j.s == total && nbuf > 0;
        }
        if (tid == 0) job = j;
        lds_barrier();
    }
    const int p = __builtin_amdgcn_readfirstlane(job.p), s = __builtin_amdgcn_readfirstlane(job.s);
    if (p < 0 || s >= ws.max_splits) return;
    const int w = __builtin_amdgcn_readfirstlane(job.w), e0 = __builtin_amdgcn_readfirstlane(job.e0);
    const int estride = __builtin_amdgcn_readfirstlane(job.stride), nbk = __builtin_amdgcn_readfirstlane(job.cnt);
    const int Lp = __builtin_amdgcn_readfirstlane(job.L);
    const int nbuf = Lp % SEG - (Lp % SEG >= UBUF ? UBUF : 0);
    int32_t *tag = ws.tag + (uint64_t)p * (ws.tag_stride / 4);
    float *part = ws.part + (uint64_t)p * (ws.part_stride / 4) + (uint64_t)s * GP * (D + 2);
    const bool is_buf = w == -2 && job.buf != 0;
    if (w == -2 && !is_buf) {
        if (tid == 0) tag[s] = -2;
        return;
    }
    const int G = g.G;

    if (is_buf) {
        // update-buffer tokens: dense and unrotated (Sec. 5.3), fp32 on the
        // vector ALU.  Logits: four lanes per token, 32 channels each, whole
        // 16-byte loads; sums: a thread per channel, eight rows per round trip.
        static_assert(NWV == 2, "128 threads: 32 tokens x 4 quarters, 128 channels");
        float *qsb = (float *)wbase;                        // [D][GP]
        float *zsb = qsb + D * GP;                          // [UBUF][GP]: logits, then weights
        const uint16_t *bk = g.buf_of(p), *bv = bk + UBUF * D;
        const int t = tid >> 2, qr = tid & 3;
        uint4 kr[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) kr[x] = ((const uint4 *)(bk + min(t, nbuf - 1) * D))[4 * qr + x];
        for (int i = tid; i < D * GP; i += NWV * 64) {
            const int c = i / GP, h = i % GP;
            qsb[i] = (h < G) ? h2f(qraw[((uint64_t)p * G + h) * D + c], g.dtype) : 0.0f;
        }
        lds_barrier();
        float z[GP];
#pragma unroll
        for (int h = 0; h < GP; ++h) z[h] = 0.0f;
        // (eight heads: a piece at a time, all of a row's reads of q at once would spill)
#pragma unroll (GP == 8 ? 1 : 4)
        for (int x = 0; x < 4; ++x) {
            const uint32_t w4[4] = {kr[0].x, kr[0].y, kr[0].z, kr[0].w};
            kr[0] = kr[1]; kr[1] = kr[2]; kr[2] = kr[3];    // (a runtime index would put them in memory)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float kv = h2f_t<DT>((e & 1) ? (w4[e >> 1] >> 16) : (w4[e >> 1] & 0xffffu));
                const float *qc = qsb + (32 * qr + 8 * x + e) * GP;
#pragma unroll
                for (int h = 0; h < GP; ++h) z[h] = fmaf(qc[h], kv, z[h]);
            }
        }
#pragma unroll
        for (int h = 0; h < GP; ++h) {
            z[h] += dpp_f<0xb1>(z[h]);                      // lanes ^ 1, then ^ 2
            z[h] += dpp_f<0x4e>(z[h]);
            if (qr == 0) zsb[t * GP + h] = t < nbuf ? z[h] * scale : -INFINITY;
        }
        lds_barrier();
        if (tid < GP) {                                     // a head's maximum, weights and sum
            float m = -INFINITY, l = 0.0f;
            for (int i = 0; i < nbuf; ++i) m = fmaxf(m, zsb[i * GP + tid]);
            for (int i = 0; i < nbuf; ++i) {
                const float e = __expf(zsb[i * GP + tid] - m);
                zsb[i * GP + tid] = e;
                l += e;
            }
            part[tid] = m;
            part[GP + tid] = l;
        }
        float ba[GP];
#pragma unroll
        for (int h = 0; h < GP; ++h) ba[h] = 0.0f;
        uint16_t vr[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) vr[x] = bv[min(x, nbuf - 1) * D + tid];
        lds_barrier();
        for (int i0 = 0; i0 < nbuf; i0 += 8) {
            float vv[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                vv[x] = h2f_t<DT>(vr[x]);
                vr[x] = bv[min(i0 + 8 + x, nbuf - 1) * D + tid];
            }
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (i0 + x < nbuf) {
#pragma unroll
                    for (int h = 0; h < GP; ++h) ba[h] = fmaf(zsb[(i0 + x) * GP + h], vv[x], ba[h]);
                }
        }
#pragma unroll
        for (int h = 0; h < GP; ++h) part[2 * GP + h * D + tid] = ba[h];
        if (tid == 0) tag[s] = -1;
        return;
    }

    // ---- split setup: one thread per selected block; blocks ordered by size
    // (16, then 8, then 4; ascending index inside a size), so every block
    // starts at a multiple of its size and none straddles a 64-token chunk
    bool all16;                                     // every record of the split 4-byte aligned (granule loads)
    bool dense = false;                             // every block keeps all D channels (RMAX = D kernels)
    int rsplit;                                     // largest kept count in the split
    {
        const bool on = tid < nbk;
        uint32_t goff = 0; int r = 0, l2g = 0, l2b = 2;
        if (on) {                                   // the entry's record offset and strategy (top-k wrote them)
            const uint2 si = ws.selinfo[(uint64_t)p * (ws.selinfo_stride / 8) + e0 + tid * estride];
            r = (int)((si.y >> 8) & 0xffu); l2g = (int)((si.y >> 16) & 3u); l2b = (int)min(max((si.y >> 20) & 7u, 2u), 4u);
            goff = min(si.x, (uint32_t)g.tok_size(p));     // keeps every read inside the arena
        }
        const int cls = on ? 4 - l2b : 3;
        const uint64_t m0 = __ballot(cls == 0), m1 = __ballot(cls == 1), m2 = __ballot(cls == 2);
        if (lane == 0) {
            wcnt[wave * 4 + 0] = __popcll(m0);
            wcnt[wave * 4 + 1] = __popcll(m1);
            wcnt[wave * 4 + 2] = __popcll(m2);
        }
        const int rw = wave_max_i(on ? r : 0);
        if (lane == 0) wcnt[wave * 4 + 3] = rw;
        // granule loads take a fixed 16-byte bitmap and whole 16-byte runs of
        // values at any 4-byte aligned record (what lies past a record is read
        // inside the arena's slack and never used; a walk reads D / g bits)
        all16 = __syncthreads_and(!on || ((goff & 3u) == 0 && (bm_bytes(l2g, g.trunc) & 3) == 0));
        if (RMAX == 0) dense = true;
        else if (RMAX >= D && !F8) dense = __syncthreads_and(!on || (l2g == 0 && r == D && (goff & 15u) == 0));
        if (on) {
            const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
            int c16 = 0, c8 = 0, before = 0;
#pragma unroll
            for (int x = 0; x < NWV; ++x) {
                c16 += wcnt[x * 4];
                c8 += wcnt[x * 4 + 1];
                before += x < wave ? wcnt[x * 4 + cls] : 0;
            }
            const int base = cls == 0 ? 0 : (cls == 1 ? c16 : c16 + c8);
            const uint64_t mc = cls == 0 ? m0 : (cls == 1 ? m1 : m2);
            const int pos = base + before + __popcll(mc & below);
            blk[pos] = make_uint2(goff, ((uint32_t)r << 8) | ((uint32_t)l2g << 16) | ((uint32_t)l2b << 20));
        }
    }
    // q operand: B[k = channel][n] of the logits K . q^T.  Column n < GP holds
    // the 16-bit high part of head n's query, column GP + n its residual, so
    // one product gives both halves of every head's logit (added across the
    // lanes afterwards): the matrix-core columns past the group are not idle.
    static_assert(2 * GP <= 16, "high and low query parts share the 16 columns");
    M8 qhl[4];
    {
        const int qw = g.rotated ? w : 0;
        const float *src = ws.qrot + (uint64_t)p * (ws.qrot_stride / 4) + (uint64_t)qw * D * GP;
        const int hq = l16 < GP ? l16 : l16 - GP;           // head of this column
        const bool live = l16 < 2 * GP && hq < G;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            float xs[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = ks * 32 + q4 * 8 + i;
                xs[i] = live ? src[c * GP + hq] : 0.0f;
            }
            M8 hi, lo;
            split8<DT>(xs, hi, lo);
            qhl[ks] = (l16 < GP) ? hi : lo;
        }
    }
    __syncthreads();
    // uniform counts (scalar registers)
    int n16 = 0, n8 = 0, n4 = 0;
    rsplit = 0;
#pragma unroll
    for (int x = 0; x < NWV; ++x) {
        n16 += wcnt[x * 4]; n8 += wcnt[x * 4 + 1]; n4 += wcnt[x * 4 + 2]; rsplit = max(rsplit, wcnt[x * 4 + 3]);
    }
    n16 = __builtin_amdgcn_readfirstlane(n16);
    n8 = __builtin_amdgcn_readfirstlane(n8);
    n4 = __builtin_amdgcn_readfirstlane(n4);
    rsplit = __builtin_amdgcn_readfirstlane(rsplit);
    const int T16 = 16 * n16, T8 = T16 + 8 * n8, T = T8 + 4 * n4;
    const int nch = (T + CH_TOK - 1) / CH_TOK;
    const uint8_t *tokg = g.tok_of(p);

    // token t of the split's ordered run -> its packed records
    auto locate = [&](int c) {
        TokLoc L;
        const int t = c * CH_TOK + lane;
        L.valid = c < nch && t < T;
        int bi, j;
        if (t < T16) { bi = t >> 4; j = t & 15; }
        else if (t < T8) { bi = n16 + ((t - T16) >> 3); j = (t - T16) & 7; }
        else { bi = n16 + n8 + ((t - T8) >> 2); j = (t - T8) & 3; }
        if (!L.valid) { bi = 0; j = 0; }
        const BlkInfo b = blk[bi];
        L.base = b.x;
        L.info = (uint32_t)j | (L.valid ? b.y : (b.y & ~0xff00u));
        return L;
    };

    float m_run = -INFINITY, l_run = 0.0f;                  // head l16
    floatx4 acc_o[8];                                       // [channel tile][head 4*q4 + r]
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) acc_o[ct] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

    // the chunk loop, compiled for aligned records (a fixed number RL of 16-byte
    // value loads per vector: 4 when no kept count of the split exceeds 32) and
    // for any records (dword loads): one straight-line load form per copy keeps
    // the prefetched registers free of copies at joins, which would wait on them
    auto chunks = [&](auto rlc) {
        constexpr int RL = decltype(rlc)::value;
        int c = wave;
        TokLoc cur = locate(c);
        using PV = std::conditional_t<F8, PVec8<RMAX>, PVec<RMAX>>;
        PV kx, vx;
        {
            const int rm = wave_max_i(cur.r());
            __builtin_amdgcn_sched_barrier(0);
            load_tok<RMAX, RL>(kx, tokg, cur, false, rm, g.trunc);
            __builtin_amdgcn_sched_barrier(0);          // K's loads before V's, as in the loop
            load_tok<RMAX, RL>(vx, tokg, cur, true, rm, g.trunc);
            __builtin_amdgcn_sched_barrier(0);
        }
        // the tile starts zero; every MFMA operand read below zeroes what it
        // read, and the reads cover every position a scatter can write, so
        // each scatter finds the tile zero again
        {
            uint4 *t4 = (uint4 *)tile;
            const uint4 zz = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int k = 0; k < TILE_BYTES / 16 / 64; ++k) t4[lane + k * 64] = zz;
        }
        wave_sync();
        for (; c < nch; c += NWV) {
            const int ntok = min(CH_TOK, T - c * CH_TOK);
            const TokLoc nxt = locate(c + NWV);
            const int rmn = wave_max_i(nxt.r());
            // ---- K: expand packed keys (token-major rows), logits on MFMA
            if (cur.valid) {
                if (g.trunc < D) mask_words(kx.bw, g.trunc >> cur.l2g());
                scatter_rec<DT, RMAX, RL, false, FR>(kx, cur.r(), cur.l2g(), lds_addr(tile) + lane * (KT_STRIDE * 2));
            }
            wave_sync();
            mem_fence_compiler();
            load_tok<RMAX, RL>(kx, tokg, nxt, false, rmn, g.trunc);
            float z[4][4];
            {
                // four independent accumulators (token groups n), so no
                // product waits on the one before it
                const uint32_t tb = lds_addr(tile);
                floatx4 a4[4];
#pragma unroll
                for (int n = 0; n < 4; ++n) a4[n] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    M8 a[4];
#pragma unroll
                    for (int n = 0; n < 4; ++n) {
                        const uint32_t ad = tb + (uint32_t)(((n * 16 + l16) * KT_STRIDE + ks * 32 + q4 * 8) * 2);
                        a[n] = __builtin_bit_cast(M8, lds_ld<u32x4>(ad));
                        lds_st<u32x4>(ad, u32x4{0u, 0u, 0u, 0u});
                    }
#pragma unroll
                    for (int n = 0; n < 4; ++n) a4[n] = Mma<DT>::run(a[n], qhl[ks], a4[n]);
                }
                // head l16 < GP: high-part logit + residual logit of column l16 + GP
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r) z[n][r] = (a4[n][r] + dpp_f<0x100 + GP>(a4[n][r])) * scale;
            }
            if (ntok < CH_TOK) {                                  // the split's last chunk
#pragma unroll
                for (int n = 0; n < 4; ++n)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (n * 16 + q4 * 4 + r >= ntok) z[n][r] = -INFINITY;
            }
            // ---- online softmax for head l16 (tokens across r, n and the lane quarters)
            float cm = -INFINITY;
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) cm = fmaxf(cm, z[n][r]);
            cm = xor_max<16>(cm);
            cm = xor_max<32>(cm);
            // every chunk holds a valid token, so mn is finite: exp(-inf - mn) = 0
            // covers the masked tokens and the first chunk's alpha
            const float mn = fmaxf(m_run, cm);
            const float alpha = __expf(m_run - mn);
            float ls = 0.0f;
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    z[n][r] = __expf(z[n][r] - mn);
                    ls += z[n][r];
                }
            ls = xor_sum<16>(ls);
            ls = xor_sum<32>(ls);
            l_run = l_run * alpha + ls;
            m_run = mn;
            // ---- V: expand packed values (channel-major rows)
            wave_sync();
            if (cur.valid) {
                if (g.trunc < D) mask_words(vx.bw, g.trunc >> cur.l2g());
                scatter_rec<DT, RMAX, RL, true, FR>(vx, cur.r(), cur.l2g(), lds_addr(tile) + lane * 2);
            }
            wave_sync();
            mem_fence_compiler();
            load_tok<RMAX, RL>(vx, tokg, nxt, true, rmn, g.trunc);
            // ---- P . V on MFMA: A = P[head l16][tokens], B = V[tokens][channel tile]
            if (!__all(alpha == 1.0f)) {                      // some head's running max moved
                float ar[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {                  // alpha of head (q4 * 4 + r) % GP
                    const float a0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha), r));
                    if (GP == 4) {
                        ar[r] = a0;
                    } else {
                        const float a1 =
                            __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, alpha), 4 + r));
                        ar[r] = (q4 & 1) ? a1 : a0;
                    }
                }
#pragma unroll
                for (int ct = 0; ct < 8; ++ct)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc_o[ct][r] *= ar[r];
            }
            const uint32_t tb = lds_addr(tile);
#pragma unroll
            for (int kv = 0; kv < 2; ++kv) {
                float xs[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) xs[i] = z[2 * kv + (i >> 2)][i & 3];
                // A rows n < GP: P's 16-bit high part for head n; rows GP + n:
                // its residual, moved over from lane n (one product for both)
                M8 ah, al;
                split8<DT>(xs, ah, al);
                u32x4 alw = __builtin_bit_cast(u32x4, al), ahw = __builtin_bit_cast(u32x4, ah);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t sh = dpp_u<0x110 + GP, 0xf>(alw[e]);
                    ahw[e] = (l16 < GP) ? ahw[e] : sh;
                }
                const M8 apl = __builtin_bit_cast(M8, ahw);
                M8 bv[8];
#pragma unroll
                for (int ct = 0; ct < 8; ++ct) {
                    const uint32_t ad = tb + (uint32_t)(((ct * 16 + l16) * VT_STRIDE + kv * 32 + q4 * 4) * 2);
                    const u32x2 v0 = lds_ld<u32x2>(ad), v1 = lds_ld<u32x2>(ad + 32);
                    lds_st<u32x2>(ad, u32x2{0u, 0u});
                    lds_st<u32x2>(ad + 32, u32x2{0u, 0u});
                    bv[ct] = __builtin_bit_cast(M8, u32x4{v0.x, v0.y, v1.x, v1.y});
                }
#pragma unroll
                for (int ct = 0; ct < 8; ++ct) acc_o[ct] = Mma<DT>::run(apl, bv[ct], acc_o[ct]);
            }
            wave_sync();
            cur = nxt;
        }
    };
    // blocks that keep every channel: their records hold dense rows, taken in
    // 32-token steps as the dense kernel takes its rows (K straight into
    // operands, V by direct loads into the tile's place, two buffers)
    auto dense_steps = [&] {
        typedef __attribute__((address_space(3))) uint8_t lds_b;
        typedef __attribute__((address_space(1))) const uint8_t gl_b;
        constexpr uint32_t VBUF = DSTEP * D * 2;
        static_assert(2 * VBUF <= TILE_BYTES, "two V buffers in a wave's tile");
        // the K (V) row of the split's token t, 256 bytes
        auto row = [&](int t, bool V_) {
            if (t >= T) t = 0;                              // (past the last token: weight zero)
            int bi, j;
            if (t < T16) { bi = t >> 4; j = t & 15; }
            else if (t < T8) { bi = n16 + ((t - T16) >> 3); j = (t - T16) & 7; }
            else { bi = n16 + n8 + ((t - T8) >> 2); j = (t - T8) & 3; }
            const BlkInfo b = blk[bi];
            const uint32_t B = 1u << ((b.y >> 20) & 7u);
            return tokg + b.x + (V_ ? B * (32 + 2 * D) : B * 16) + (uint32_t)j * (2 * D);
        };
        auto load_k = [&](int t, uint4 (&x)[2][4]) {
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const uint4 *r = (const uint4 *)row(t + 16 * n + l16, false) + q4;
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) x[n][ks] = r[4 * ks];
            }
        };
        auto load_v = [&](int t, int buf) {
#pragma unroll
            for (int i = 0; i < DSTEP / 4; ++i) {
                const int r = 4 * i + q4;
                __builtin_amdgcn_global_load_lds((gl_b *)(row(t + r, true) + 16 * (l16 ^ (r & 15))),
                                                 (lds_b *)(tile + buf * VBUF + 1024 * i), 16, 0, 0);
            }
        };
        uint32_t va[8];
        tr_addresses(lds_addr(tile), va);
        int t = DSTEP * wave;
        auto step = [&](const uint4 (&kx)[2][4], uint4 (&kn)[2][4], const int buf) {
            const int tn = t + DSTEP * NWV < T ? t + DSTEP * NWV : t;
            __builtin_amdgcn_sched_barrier(0);
            load_k(tn, kn);
            __builtin_amdgcn_sched_barrier(0);              // K's loads before V's: the wait below counts on it
            load_v(tn, buf ^ 1);
            __builtin_amdgcn_sched_barrier(0);
            float z[2][4];
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                floatx4 a = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) a = Mma<DT>::run(__builtin_bit_cast(M8, kx[n][ks]), qhl[ks], a);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    z[n][r] = (a[r] + dpp_f<0x100 + GP>(a[r])) * scale;
                    if (t + 16 * n + 4 * q4 + r >= T) z[n][r] = -INFINITY;
                }
            }
            dense_accumulate<DT, GP, 2>(z, m_run, l_run, acc_o, 1.0f, [&] {
                // this step's V rows have landed once only the next step's 8 + 8 loads are out
                asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
            }, va, buf * VBUF);
            t += DSTEP * NWV;
        };
        uint4 k0[2][4], k1[2][4];
        if (t < T) { load_k(t, k0); load_v(t, 0); }
        while (t < T) {
            step(k0, k1, 0);
            if (t >= T) break;
            step(k1, k0, 1);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // (the merge reuses the buffers)
    };
    bool done = false;
    if constexpr (RMAX == 0) {
        dense_steps();
        done = true;
    } else if constexpr (RMAX >= D && !F8) {
        if (all16 && dense) { dense_steps(); done = true; }
    }
    if constexpr (RMAX > 0) if (!done) {
        if (!all16) chunks(IntC<0>{});
        else if (RMAX > 32 && rsplit <= 32) chunks(IntC<4>{});
        else chunks(IntC<RMAX / 8>{});
    }
    // ---- merge the waves' (m, l, acc) and write the split's partial
    lds_barrier();
    float *mrg = (float *)(wbase + wave * TILE_BYTES);      // [16][D + 2]
    if (q4 == 0) { mrg[l16 * (D + 2)] = m_run; mrg[l16 * (D + 2) + 1] = l_run; }
#pragma unroll
    for (int ct = 0; ct < 8; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r) mrg[(q4 * 4 + r) * (D + 2) + 2 + ct * 16 + l16] = acc_o[ct][r];
    lds_barrier();
    // the merged (max, sum, accumulator) of the split, in the window's rotated
    // space (the combine rotates each window's sum back once)
    for (int i = tid; i < GP * D; i += NWV * 64) {
        const int h = i / D, cc = i % D;
        float Mx = -INFINITY;
#pragma unroll
        for (int x = 0; x < NWV; ++x) Mx = fmaxf(Mx, ((const float *)(wbase + x * TILE_BYTES))[h * (D + 2)]);
        float A = 0.0f, Ls = 0.0f;
#pragma unroll
        for (int x = 0; x < NWV; ++x) {
            const float *mw = (const float *)(wbase + x * TILE_BYTES);
            const float f = (mw[h * (D + 2)] == -INFINITY) ? 0.0f : __expf(mw[h * (D + 2)] - Mx);
            A += (mw[h * (D + 2) + 2 + cc] + mw[(h + GP) * (D + 2) + 2 + cc]) * f;   // high + residual rows
            Ls += mw[h * (D + 2) + 1] * f;
        }
        part[2 * GP + h * D + cc] = A;
        if (cc == 0) { part[h] = Mx; part[GP + h] = Ls; }
    }
    if (tid == 0) tag[s] = w;
}

template <int DT, int GP>
hipError_t attn_dt(const Geom &g, const WsGeom &w, float scale, const uint16_t *q, bool fixed, bool small, hipStream_t s) {
    // Workgroups past the last split derive the plan and end, so the grid is no
    // larger than the plan that the kernel takes can need.  The register plan
    // has as many splits as whole rounds of the resident workgroups, the general
    // one as fill a single round or as splits of SPLIT_MAX blocks, both with one
    // rounding split more per window and buffer; and never more than the most
    // blocks that can be selected in splits of the plan's least size, or than
    // every pair's whole partial array.  (Sized by rounds for both, and by a round
    // more than needed, one sequence of 60000 tokens beside 31 of 500 launched
    // 7680 workgroups of the general plan, 82 us in this kernel; 3584 take 46.)
    const size_t smem = ATTN_HDR_BYTES + (size_t)ATTN_NWV * TILE_BYTES;
    const long long extra = (long long)g.npairs * (g.nw + 1);
    const long long most = (long long)g.npairs * ceil_div(w.max_sel, SPLIT_MAX);
    const long long room = std::max<long long>(std::max<long long>(w.split_slots - extra, w.split_slots / 4), 1);    // (the plan's, at least)
    const long long whole = register_plan(g) ? (most + room - 1) / room * w.split_slots : std::max<long long>(w.split_slots, most);
    const long long least = (long long)g.npairs * ceil_div(w.max_sel, register_plan(g) ? SPLIT_LEAST : SPLIT_MIN);
    const long long nwg = std::min<long long>(std::min(whole, least) + extra, (long long)g.npairs * w.max_splits);
    const unsigned grid = w.fix_splits ? (unsigned)(g.npairs * (w.fix_splits + 1)) : (unsigned)nwg;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * ATTN_NWV), smem, s, g, w, scale, q);
        return hipGetLastError();
    };
    // one strategy that keeps every channel: no record needs a walk
    if (g.force && g.def_keep == D && g.def_group == 1 && !g.fp8) return go(k_attn<DT, GP, 0, false, false>);
    if (g.fp8) return fixed ? go(k_attn<DT, GP, 48, true, true>)
                            : (small ? go(k_attn<DT, GP, 48, false, true>) : go(k_attn<DT, GP, 128, false, true>));
    return fixed ? go(k_attn<DT, GP, 48, true, false>)
                 : (small ? go(k_attn<DT, GP, 48, false, false>) : go(k_attn<DT, GP, 128, false, false>));
}

}  // namespace

}  // namespace mosaic
