// decode_common.h -- shared by the decode step's kernels (score.hip, attn.h,
// decode.hip): matrix-core and LDS access helpers, lane scans, and the walk
// over packed vectors' bitmaps (not part of the C ABI).
#pragma once
#include "dense_step.h"

namespace mosaic {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 halfx8;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

template <int DT> struct Mma;
template <> struct Mma<1> {
    using v8 = bf16x8;
    using el = __bf16;
    static __device__ __forceinline__ floatx4 run(v8 a, v8 b, floatx4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    }
};
template <> struct Mma<0> {
    using v8 = halfx8;
    using el = _Float16;
    static __device__ __forceinline__ floatx4 run(v8 a, v8 b, floatx4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
    }
};

template <int DT> __device__ __forceinline__ float h2f_t(uint32_t h16) {
    if (DT) return __uint_as_float(h16 << 16);
    return (float)__builtin_bit_cast(_Float16, (uint16_t)h16);
}

__device__ __forceinline__ void wave_sync() { __builtin_amdgcn_wave_barrier(); }

// LDS byte addresses as plain integers (so that address arithmetic folds into
// single mad/shift-add instructions) and accesses through them
typedef __attribute__((address_space(3))) uint8_t lds_u8;
__device__ __forceinline__ uint32_t lds_addr(const void *p) { return (uint32_t)(uintptr_t)(const lds_u8 *)p; }
template <typename T> __device__ __forceinline__ T lds_ld(uint32_t a) {
    return *(const __attribute__((address_space(3))) T *)(uintptr_t)a;
}
template <typename T> __device__ __forceinline__ void lds_st(uint32_t a, T v) {
    *(__attribute__((address_space(3))) T *)(uintptr_t)a = v;
}
// keep the compiler from moving memory operations across this point
__device__ __forceinline__ void mem_fence_compiler() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ int pair_ndesc(const PairMeta &m, int &n_final, int &prov, int &nbuf) {
    n_final = m.L / SEG;
    const int rem = m.L % SEG;
    prov = rem >= UBUF;
    nbuf = rem - (prov ? UBUF : 0);
    return n_final + prov;
}

__device__ __forceinline__ int pair_nblocks(const Geom &g, int p, const PairMeta &m) {
    int nf, prov, nbuf;
    pair_ndesc(m, nf, prov, nbuf);
    int nb = m.nblk_final;
    if (prov) nb += UBUF >> g.desc_of(p)[nf].log2b;
    return nb;
}

// Copy nbytes (multiple of 16) from global to LDS with 16-byte loads; all of
// a thread's loads are issued before its stores.
template <int NT, int MAXPER>
__device__ __forceinline__ void stage_copy(uint4 *dst, const uint4 *src, int nbytes, int tid) {
    const int n = nbytes >> 4;
    uint4 r[MAXPER];
#pragma unroll
    for (int k = 0; k < MAXPER; ++k) {
        const int i = tid + k * NT;
        if (i < n) r[k] = src[i];
        else r[k] = make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int k = 0; k < MAXPER; ++k) {
        const int i = tid + k * NT;
        if (i < n) dst[i] = r[k];
    }
}

// wave-level inclusive scans on the data-parallel-primitive lane shifts (no
// LDS round trips): shifts by 1, 2, 4, 8 inside each 16-lane row, then the
// row broadcasts of lanes 15 and 31
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_u(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}
// x combined with its value in lane ^ 16 or lane ^ 32, on the cross-row
// swap instructions (no LDS round trip): the swap leaves each lane holding
// its own value and its partner's
template <int X>
__device__ __forceinline__ void xor_pair(float x, float &a, float &b) {
    static_assert(X == 16 || X == 32, "row pairs or wave halves");
    const uint32_t u = __float_as_uint(x);
    if (X == 16) { const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false); a = __uint_as_float(r[0]); b = __uint_as_float(r[1]); }
    else { const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false); a = __uint_as_float(r[0]); b = __uint_as_float(r[1]); }
}
template <int X> __device__ __forceinline__ float xor_max(float x) { float a, b; xor_pair<X>(x, a, b); return fmaxf(a, b); }
template <int X> __device__ __forceinline__ float xor_sum(float x) { float a, b; xor_pair<X>(x, a, b); return a + b; }

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t x) {
    x += dpp_u<0x111, 0xf>(x);
    x += dpp_u<0x112, 0xf>(x);
    x += dpp_u<0x114, 0xf>(x);
    x += dpp_u<0x118, 0xf>(x);
    x += dpp_u<0x142, 0xa>(x);
    x += dpp_u<0x143, 0xc>(x);
    return x;
}
// maximum over the wave (every lane active); lanes that read out of range get 0
__device__ __forceinline__ uint32_t wave_max_u(uint32_t x) {
    x = max(x, dpp_u<0x111, 0xf>(x));
    x = max(x, dpp_u<0x112, 0xf>(x));
    x = max(x, dpp_u<0x114, 0xf>(x));
    x = max(x, dpp_u<0x118, 0xf>(x));
    x = max(x, dpp_u<0x142, 0xa>(x));
    x = max(x, dpp_u<0x143, 0xc>(x));
    return (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
}

// ------------------------------------------------------------------ bitmap walk
// A packed vector keeps r values in ascending channel order; its bitmap marks
// the kept groups of 1 << log2g channels.  The walk visits the set bits in
// ascending order, one per step, so that a fixed, unrolled slot sequence can
// take the values from registers.  The position is v_ffbl of the current
// bitmap word; the words are walked in order, with empty words in the middle
// squeezed out first so that a step moves on by at most one word.  Each word
// carries the caller's address of its first group.
struct Walk {
    uint32_t cur, n1, n2, n3;
    uint32_t a, a1, a2, a3;
    __device__ __forceinline__ uint32_t pos() const { return (uint32_t)__builtin_ctz(cur); }
    template <int NWD>
    __device__ __forceinline__ void step() {
        cur &= cur - 1u;
        if (NWD > 1) {
            const bool z = cur == 0u;
            cur = z ? n1 : cur;
            a = z ? a1 : a;
            if (NWD > 2) {
                n1 = z ? n2 : n1; a1 = z ? a2 : a1;
                n2 = z ? n3 : n2; a2 = z ? a3 : a2;
            }
        }
    }
};

__device__ __forceinline__ void cswap_empty(uint32_t &wa, uint32_t &aa, uint32_t &wb, uint32_t &ab) {
    const bool z = wa == 0u;
    wa = z ? wb : wa;
    aa = z ? ab : aa;
    wb = z ? 0u : wb;
}

template <int NWD>
__device__ __forceinline__ Walk make_walk(const uint32_t (&bw)[4], uint32_t a0, uint32_t astep) {
    uint32_t w[4], a[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) { w[k] = k < NWD ? bw[k] : 0u; a[k] = a0 + (uint32_t)k * astep; }
    if (NWD == 2) {
        const bool hole = w[0] == 0u && w[1] != 0u;
        if (__ballot(hole)) cswap_empty(w[0], a[0], w[1], a[1]);
    } else if (NWD == 4) {
        const bool hole = (w[0] == 0u && (w[1] | w[2] | w[3]) != 0u) || (w[1] == 0u && (w[2] | w[3]) != 0u) ||
                          (w[2] == 0u && w[3] != 0u);
        if (__ballot(hole)) {                      // stable: non-empty words to the front
#pragma unroll
            for (int round = 0; round < 2; ++round) {
                cswap_empty(w[0], a[0], w[1], a[1]);
                cswap_empty(w[2], a[2], w[3], a[3]);
                cswap_empty(w[1], a[1], w[2], a[2]);
            }
        }
    }
    Walk wk;
    wk.cur = w[0]; wk.n1 = w[1]; wk.n2 = w[2]; wk.n3 = w[3];
    wk.a = a[0]; wk.a1 = a[1]; wk.a2 = a[2]; wk.a3 = a[3];
    return wk;
}

// A truncated bitmap (Sec. 5.2: only the first T channels are represented)
// has T / g bits; the whole 16-byte bitmap loads read the values after it
// as well, so the words are cut to the first nbits bits before a walk.
__device__ __forceinline__ void mask_words(uint32_t (&bw)[4], int nbits) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int lo = 32 * k;
        bw[k] = nbits >= lo + 32 ? bw[k] : (nbits <= lo ? 0u : bw[k] & ((1u << (nbits - lo)) - 1u));
    }
}

// element s (static) of packed 16-bit values held two per dword
template <int N>
__device__ __forceinline__ uint32_t half_at(const uint32_t (&v)[N], int s) {
    return (s & 1) ? (v[s >> 1] >> 16) : (v[s >> 1] & 0xffffu);
}

// 16 bytes at a 4-byte aligned address: every record is 4-byte aligned, and
// the target runs vector memory loads in unaligned mode, so one dwordx4 load
// serves any record (the compiler merges plain dword runs the same way)
typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));

// N dwords starting at any byte p: the N + 1 aligned dwords that cover them,
// joined pairwise by byte shifts (v_alignbyte).  Truncated bitmaps of 3 or 6
// bytes put token bitmaps and block-key records at any byte; the one dword
// read past the end stays inside the arena's slack.
template <int N>
__device__ __forceinline__ void load_dwords_any(const uint8_t *p, uint32_t (&out)[N]) {
    const uintptr_t a = (uintptr_t)p;
    const uint32_t *b = (const uint32_t *)(a & ~(uintptr_t)3);
    const uint32_t sh = (uint32_t)(a & 3u);
    uint32_t w[N + 1];
#pragma unroll
    for (int k = 0; k <= N; ++k) w[k] = b[k];
#pragma unroll
    for (int k = 0; k < N; ++k) out[k] = __builtin_amdgcn_alignbyte(w[k + 1], w[k], sh);
}

// A packed vector (bitmap words + values) held in registers.
template <int RMAX>
struct PVec {
    uint32_t bw[4];
    uint32_t v[RMAX / 2];
};

// A token record with one-byte E4M3 values, as loaded (four codes per word,
// slot order from the low byte); widened to the dtype just before its walk,
// so that the loads of a prefetch are not waited on where they are issued.
template <int RMAX>
struct PVec8 {
    uint32_t bw[4];
    uint32_t v[RMAX / 4];
};

// codes 2 HI and 2 HI + 1 of w -> the two 16-bit values of the dtype (exact:
// every E4M3 value is a bf16 and an fp16 value), the first in the low half
template <int DT, bool HI>
__device__ __forceinline__ uint32_t e4m3x2(uint32_t w) {
    if constexpr (DT) return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, HI));
    else return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(w, 1.0f, HI));
}

// the first NW words of codes (4 NW values) widened into a 16-bit vector
template <int DT, int RMAX, int NW>
__device__ __forceinline__ void widen(const PVec8<RMAX> &c, PVec<RMAX> &x) {
    static_assert(NW <= RMAX / 4, "code words");
#pragma unroll
    for (int k = 0; k < 4; ++k) x.bw[k] = c.bw[k];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        x.v[2 * k] = e4m3x2<DT, false>(c.v[k]);
        x.v[2 * k + 1] = e4m3x2<DT, true>(c.v[k]);
    }
}

// bm and val point at the vector's bitmap and values; rmax is the largest r
// in the wave (uniform) and a16 (uniform) says both pointers are 16-byte
// aligned (A16: always so).  The loads take a fixed 16-byte bitmap and rmax
// values: what lies past a vector's own bitmap or values is read (inside the
// arena's slack) and never used.  Value slots at or past rmax keep what they
// held: a walk reads only its first r slots, and leaving them unwritten keeps
// the registers of earlier, still outstanding loads free of write-after-write
// waits.
//
// A16: 1 = the pointers are known 16-byte aligned, 0 = dword loads, -1 = chosen
// by a16 at run time.  ZF zero-fills the slots past rmax.  Without it every
// slot is loaded, those past rmax from the start of the values again (lines
// the wave reads anyway): straight-line loads with no branch, so that a
// prefetch into loop-carried registers leaves no join whose bookkeeping would
// make the wave wait on loads that are still in flight.
//
// RL > 0: exactly the first RL 16-byte granules of values and a 16-byte
// bitmap, with no condition (the caller knows r <= 8 RL for every lane of the
// wave), at any 4-byte aligned record.
template <int RMAX, int A16, bool ZF, int RL = 0>
__device__ __forceinline__ void load_pvec(PVec<RMAX> &x, const uint8_t *bm, const uint8_t *val, int rmax, bool a16) {
    static_assert(RL == 0 || (A16 == 1 && RL <= RMAX / 8), "fixed granule count");
    if (RL > 0) {
        const u32x4a4 b = *(const u32x4a4 *)bm;
        x.bw[0] = b.x; x.bw[1] = b.y; x.bw[2] = b.z; x.bw[3] = b.w;
        const u32x4a4 *v4 = (const u32x4a4 *)val;
#pragma unroll
        for (int k = 0; k < RL; ++k) {
            const u32x4a4 t = v4[k];
            x.v[4 * k] = t.x; x.v[4 * k + 1] = t.y; x.v[4 * k + 2] = t.z; x.v[4 * k + 3] = t.w;
        }
    } else if (A16 == 1 || (A16 == -1 && a16)) {
        const uint4 b = *(const uint4 *)bm;
        x.bw[0] = b.x; x.bw[1] = b.y; x.bw[2] = b.z; x.bw[3] = b.w;
        const uint4 *v4 = (const uint4 *)val;
#pragma unroll
        for (int k = 0; k < RMAX / 8; ++k) {
            uint4 t;
            if (ZF) {
                t = make_uint4(0u, 0u, 0u, 0u);
                if (8 * k < rmax) t = v4[k];
            } else {
                t = v4[(8 * k < rmax) ? k : 0];
            }
            x.v[4 * k] = t.x; x.v[4 * k + 1] = t.y; x.v[4 * k + 2] = t.z; x.v[4 * k + 3] = t.w;
        }
    } else {
        // dword loads at any byte: the bitmap, then the values below rmax
        // (those past it from the start of the values again, or zero with ZF)
        load_dwords_any<4>(bm, x.bw);
        const uintptr_t va = (uintptr_t)val;
        const uint32_t *v = (const uint32_t *)(va & ~(uintptr_t)3);
        const uint32_t sh = (uint32_t)(va & 3u);
        uint32_t u[RMAX / 2 + 1];
#pragma unroll
        for (int k = 0; k <= RMAX / 2; ++k) u[k] = v[(2 * k < rmax + 2) ? k : 0];
#pragma unroll
        for (int k = 0; k < RMAX / 2; ++k) {
            const uint32_t t = __builtin_amdgcn_alignbyte(u[k + 1], u[k], sh);
            x.v[k] = (ZF && 2 * k >= rmax) ? 0u : t;
        }
    }
}

// maximum over the wave of 0 <= v < 256 (every lane active): eight ballots,
// no cross-lane data movement
__device__ __forceinline__ int wave_max_i(int v) {
    int m = 0;
#pragma unroll
    for (int b = 7; b >= 0; --b) {
        const int c = m | (1 << b);
        if (__ballot(v >= c)) m = c;
    }
    return m;
}

template <int V> struct IntC { static constexpr int value = V; };

// Splits of a pair's one window of k selected entries under the fixed plan:
// its selected tokens in shares of split_tok, none empty, none above SPLIT_MAX
// entries.  The attention and the combine derive the same number.
__device__ __forceinline__ int fixed_splits(const Geom &g, const WsGeom &ws, int L, int k) {
    const float tok = (float)(L / UBUF * UBUF) * (float)g.sel_num / (float)g.sel_den;
    const int s = max((int)(tok / ws.split_tok) + 1, (k + SPLIT_MAX - 1) / SPLIT_MAX);
    return min(min(s, ws.fix_splits), k);
}

}  // namespace mosaic
