// Register-blocked negacyclic NTT helpers shared by the query front end and
// the ColTor stage.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>

#include "modarith.h"

namespace pir {

// Register-blocked transform for N >= 256: a polynomial is handled by
// T = N/16 threads that each keep 16 of its values in registers.  The
// butterfly stages (bit x of the pair distance, from logN-1 down to 0) run in
// chunks of up to four: during a chunk the register index r of a thread
// covers four index bits [lo, lo+4) (for the last chunk, bits [0, 4)), so
// every pair of the chunk's stages is local to one thread; between chunks
// the values are redistributed through LDS (padded one word per 16).  The
// element index of (thread t, register r) with register bits starting at lo:
//   e = (t mod 2^lo) | r << lo | (t >> lo) << (lo + 4).
// The butterfly of stage x on pair (e, e + 2^x) uses the psi power of group
// e >> (x+1) among N >> (x+1) groups, exactly as the one-stage-per-barrier
// form.  A last exchange writes point bitrev(e) so that global stores are in
// natural point order and coalesced.
//
// Register bits from lo <= 6 on leave element bits 10 and up to thread bits 6
// and up, so a wave (64 threads, 1024 elements) keeps the elements of its own
// part of the polynomial: an exchange between two such arrangements needs no
// barrier, and one into or out of them a single one (N <= 1024: none at all).
// The barriers wait for LDS only: __syncthreads() also waits for the global
// loads in flight, the next polynomial's among them.
constexpr int QR = 16;   // values per thread

__device__ __forceinline__ void lds_sync() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Orders the LDS accesses of one wave (they execute in program order; this
// keeps the compiler from reordering them).
__device__ __forceinline__ void lds_wave_order() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ uint32_t qf_pad(uint32_t e) { return e + (e >> 4); }

// Values travel in the high word of a 64-bit register pair whose low word is
// zero, the form in which v_mad_u64_u32 takes and leaves them: with the
// Montgomery form w' = w 2^32 mod q of a twiddle and -q^-1 mod 2^32,
//   p = x 2^32 + y w',  m = p (-q^-1) mod 2^32,  p + m q = (x + t) 2^32,
// t = y w mod q in [0, 2q) for any 32-bit y: three instructions for x + t, and
// x - t + 2q = 2x + 2q - (x + t) two more.  (Shoup's product and the two sums
// take six, and a companion word per twiddle.)
__device__ __forceinline__ uint32_t hi32(uint64_t v) { return (uint32_t)(v >> 32); }
__device__ __forceinline__ uint64_t with_hi(uint64_t v, uint32_t x) { return (uint64_t)x << 32 | (uint32_t)v; }

__device__ __forceinline__ void mont_bfly(uint64_t &x, uint64_t &y, uint32_t w, uint32_t q, uint32_t qn) {
    uint64_t p = (uint64_t)hi32(y) * w + x;
    p = (uint64_t)((uint32_t)p * qn) * q + p;
    y = with_hi(y, 2 * hi32(x) + 2 * q - hi32(p));
    x = p;
}

// A 64-bit sum mod q, canonical, q < 2^30: two Montgomery steps, the second by
// 2^64 mod q.  The first leaves at most hi + q + 1, so hi comes below 2q first,
// unless the caller knows that hi + q stays below 2^32 (SMALL).  r1 =
// floor(2^32 / q).  Ten instructions, seven for SMALL (a 64-bit Barrett
// reduction: about twenty).
template <bool SMALL>
__device__ __forceinline__ uint32_t mont_reduce(uint64_t x, uint32_t r64, uint32_t r1, uint32_t q, uint32_t qn) {
    if (!SMALL) x = with_hi(x, hi32(x) - __umulhi(hi32(x), r1) * q);
    const uint32_t y = hi32((uint64_t)((uint32_t)x * qn) * q + x);   // < 3q, or < 2^32
    const uint64_t z = (uint64_t)y * r64;
    const uint32_t w = hi32((uint64_t)((uint32_t)z * qn) * q + z);   // < 2q
    return min(w, w - q);
}

// x w mod q in [0, 2q), w in Montgomery form, any 32-bit x.
__device__ __forceinline__ uint32_t mont_mul(uint32_t x, uint32_t w, uint32_t q, uint32_t qn) {
    const uint64_t p = (uint64_t)x * w;
    return hi32((uint64_t)((uint32_t)p * qn) * q + p);
}

// [0, 4q) -> [0, q)
__device__ __forceinline__ uint32_t qf_reduce4(uint32_t x, uint32_t q, uint32_t q2) {
    x = min(x, x - q2);
    return min(x, x - q);
}
__device__ __forceinline__ uint32_t qf_elem(uint32_t t, uint32_t r, uint32_t lo) {
    return (t & ((1u << lo) - 1)) | (r << lo) | ((t >> lo) << (lo + 4));
}

// qf_elem(t, r, lo) is qf_elem(t, 0, lo) | r << lo with disjoint bit fields,
// so a shift, a bit reversal or the padding of it splits into a part of the
// thread and a part of the register index, which is a compile-time constant
// in the unrolled loops (qf_pad(a | b) = qf_pad(a) + qf_pad(b) for disjoint
// a and b): the LDS exchanges, twiddle reads and stores then take a per-
// thread base and immediate offsets instead of recomputing the index of
// every register (those index computations were a quarter of the
// transform's vector instructions).
__device__ __forceinline__ uint32_t qf_rpart(int r, uint32_t lo) { return (uint32_t)r << lo; }

// Butterfly forms of ntt_reg_block.
enum : int {
    NTT_LAZY = 0,   // q < 2^30: values in [0, 4q), x brought below 2q before each butterfly
    NTT_WIDE = 1,   // q >= 2^30: canonical, 64-bit intermediates, values in [0, q)
    NTT_GROW = 2,   // (1 + 2 logN) q < 2^32: no correction at all, (x + t, x - t + 2q)
};

// A value of the transform: a pair as above, one word in the wide form.
template <int MODE>
using NttVal = std::conditional_t<MODE == NTT_WIDE, uint32_t, uint64_t>;
__device__ __forceinline__ uint32_t ntt_get(uint32_t v) { return v; }
__device__ __forceinline__ uint32_t ntt_get(uint64_t v) { return hi32(v); }
__device__ __forceinline__ void ntt_set(uint32_t &v, uint32_t x) { v = x; }
__device__ __forceinline__ void ntt_set(uint64_t &v, uint32_t x) { v = with_hi(v, x); }

// Twiddle sources of ntt_reg_block: tw(x, gi) returns the psi power of group
// index gi (used by stage x), in Montgomery form, or for NTT_WIDE plain with
// its Shoup companion.
struct TwGlobal {   // tables in global memory (w: plain or Montgomery form)
    const uint32_t *w, *ws;
    __device__ __forceinline__ uint2 operator()(int, uint32_t gi) const { return make_uint2(w[gi], ws[gi]); }
};

// Twiddles staged in LDS (tw_lds_fill).  Stage x uses the groups
// [N >> (x+1), N >> x); in the last chunk (register bits from 0, element
// r | 16t) thread t needs groups (N >> (x+1)) + t K + k, k < K = 2^(3-x), of
// stages x <= 3.  Those are stored at (N >> (x+1)) + k N/16 + t, so that the
// lanes of a wave read consecutive words instead of words K apart (K-way bank
// conflicts); the slot of a group depends on the group alone, so other
// chunks' reads of these stages stay correct.
template <int LOGN>
__host__ __device__ __forceinline__ uint32_t tw_slot(int x, uint32_t gi) {
    constexpr uint32_t n = 1u << LOGN, T = n / QR;
    if (x > 3) return gi;
    const uint32_t base = n >> (x + 1), j = gi - base, sh = 3 - (uint32_t)x;
    return base + (j & ((1u << sh) - 1)) * T + (j >> sh);
}

template <int LOGN, bool PAIRS>   // PAIRS: the companions behind the N words
struct TwLds {
    const uint32_t *p;
    __device__ __forceinline__ uint2 operator()(int x, uint32_t gi) const {
        const uint32_t i = tw_slot<LOGN>(x, gi);
        return make_uint2(p[i], PAIRS ? p[(1u << LOGN) + i] : 0);
    }
};

// Fills the words of TwLds from an NttTables' fwd (the N/16 threads of a group,
// thread t); the caller synchronises before use.
template <int LOGN, bool PAIRS>
__device__ __forceinline__ void tw_lds_fill(uint32_t *p, const uint32_t *fwd, uint32_t t) {
    constexpr uint32_t n = 1u << LOGN, T = n / QR;
    const uint4 *src = reinterpret_cast<const uint4 *>(fwd + (PAIRS ? 3 : 5) * n);
#pragma unroll
    for (uint32_t i = 0; i < (PAIRS ? 8 : 4); ++i) reinterpret_cast<uint4 *>(p)[t + i * T] = src[t + i * T];
}

// The up to 15 twiddles that a thread needs for the stages [clo, hi) of a chunk
// with register bits from lo: stage lo + b uses 2^(3-b), at [2^(3-b) - 1 + k]
// the one of registers k 2^(b+1) .. (k+1) 2^(b+1) - 1.
template <int LOGN, class TW>
__device__ __forceinline__ void tw_chunk(uint2 (&w)[QR], uint32_t t, int lo, int clo, int hi, const TW &tw) {
    constexpr uint32_t n = 1u << LOGN;
#pragma unroll
    for (int x = hi - 1; x >= clo; --x) {
        const int b = x - lo;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (k < 8 >> b)
                w[(8 >> b) - 1 + k] =
                    tw(x, (n >> (x + 1)) + (qf_elem(t, (uint32_t)k << (b + 1), (uint32_t)lo) >> (x + 1)));
    }
}

// Those of the first chunk are the same for every thread: in scalar registers,
// for as many transforms as the caller makes.
template <int LOGN, class TW>
__device__ __forceinline__ void tw_first(uint2 (&w)[QR], const TW &tw) {
    tw_chunk<LOGN>(w, 0, LOGN - 4, LOGN - 4, LOGN, tw);
#pragma unroll
    for (int k = 0; k + 1 < QR; ++k)
        w[k] = make_uint2(__builtin_amdgcn_readfirstlane(w[k].x), __builtin_amdgcn_readfirstlane(w[k].y));
}

// Forward transform of one polynomial held by N/16 threads (N = 2^LOGN >=
// 256).  On entry register r of thread t holds element qf_elem(t, r, LOGN - 4)
// of the natural coefficient order (a residue below q); on return it holds
// element 16t + r of the transform, which is point bitrev(16t + r), congruent
// mod q and bounded by the form: NTT_WIDE [0, q), NTT_LAZY [0, 4q), NTT_GROW
// [0, (1 + 2 logN) q) (each stage adds at most 2q).  poly is LDS of N + N/16
// words that no other wave reads any more; on return a wave has read only its
// own 1024 elements' part since the last barrier.  w0: tw_first's; tw: the
// twiddle source of the later chunks, each chunk's read before the exchange
// that leads to it (read one by one at their butterflies, the waits for LDS
// took longer than the butterflies of a lone wave); qn: -q^-1 mod 2^32 (not
// used by NTT_WIDE); last: called before the last exchange, for loads that are
// to arrive during the last butterflies.
template <int LOGN, int MODE, class TW, class LAST>
__device__ __forceinline__ void ntt_reg_block(NttVal<MODE> (&v)[QR], uint32_t t, uint32_t *poly,
                                              const uint2 (&w0)[QR], const TW &tw, uint32_t q, uint32_t qn,
                                              LAST &&last) {
    int lo = LOGN - 4;
    uint2 w[QR];
#pragma unroll
    for (int k = 0; k + 1 < QR; ++k) w[k] = w0[k];
#pragma unroll
    for (int hi = LOGN; hi > 0; hi -= 4) {
        const int clo = hi - 4 > 0 ? hi - 4 : 0;
        if (hi < LOGN) {
            const uint32_t pw = qf_pad(qf_elem(t, 0, lo)), pr = qf_pad(qf_elem(t, 0, clo));
#pragma unroll
            for (int r = 0; r < QR; ++r) poly[pw + qf_pad(qf_rpart(r, lo))] = ntt_get(v[r]);
            tw_chunk<LOGN>(w, t, clo, clo, hi, tw);
            if (clo == 0) last();
            if (lo > 6) lds_sync();
            else lds_wave_order();
#pragma unroll
            for (int r = 0; r < QR; ++r) ntt_set(v[r], poly[pr + qf_pad(qf_rpart(r, clo))]);
            if (lo <= 6) lds_wave_order();
            lo = clo;
        }
#pragma unroll
        for (int x = hi - 1; x >= clo; --x) {
            const int b = x - lo, bit = 1 << b;
#pragma unroll
            for (int r = 0; r < QR; ++r) {
                if (r & bit) continue;
                const uint2 w2 = w[(8 >> b) - 1 + (r >> (b + 1))];
                if constexpr (MODE == NTT_WIDE) {
                    const uint32_t u = v[r], y = mul_shoup_w(v[r | bit], w2.x, w2.y, q);
                    v[r] = add_mod_w(u, y, q);
                    v[r | bit] = sub_mod(u, y, q);
                } else {
                    if (MODE == NTT_LAZY) v[r] = with_hi(v[r], min(hi32(v[r]), hi32(v[r]) - 2 * q));
                    mont_bfly(v[r], v[r | bit], w2.x, q, qn);
                }
            }
        }
    }
}

// Inverse transform by decimation in time, with the butterfly of the forward
// one: the plain discrete Fourier transform of bit-reversed input, whose first
// two stages need no product for the power 1, and the powers of psi^-1 left to
// the caller's scaling (merged into Gentleman-Sande butterflies, whose sums
// need a correction of their own, they take eight instructions a butterfly).
// On entry register r of thread t holds position 16t + r of the bit-reversed
// arrangement (point bitrev(16t + r)), a residue below q; on return N psi^i
// times coefficient i = qf_elem(t, r, LOGN - 4), bounded as for
// ntt_reg_block.  w: Montgomery forms of omega^-(k N / 2^(s+1)) at 2^s + k for
// stage s, k < 2^s (omega = psi^2).  poly as for intt_reg_block.
template <int LOGN, int MODE>
__device__ __forceinline__ void intt_dit_block(uint64_t (&v)[QR], uint32_t t, uint32_t *poly, const uint32_t *w,
                                               uint32_t q, uint32_t qn) {
    static_assert(MODE != NTT_WIDE, "");
    int lo = 0;
#pragma unroll
    for (int clo = 0; clo < LOGN; clo += 4) {
        const int chi = clo + 4 < LOGN ? clo + 4 : LOGN;
        const int rlo = clo < LOGN - 4 ? clo : LOGN - 4;   // registers cover [rlo, rlo + 4)
        uint32_t tw[QR];   // stage rlo + b: the power of registers = k mod 2^b at 2^b - 1 + k
        const uint32_t tl = t & ((1u << rlo) - 1);
#pragma unroll
        for (int s = clo; s < chi; ++s) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k < 1 << (s - rlo)) tw[(1 << (s - rlo)) - 1 + k] = (w + (1u << s) + ((uint32_t)k << rlo))[tl];
        }
        if (rlo != lo) {
            if (lo > 6) lds_sync();   // the other waves have read what this one overwrites
            else lds_wave_order();
            const uint32_t pw = qf_pad(qf_elem(t, 0, lo)), pr = qf_pad(qf_elem(t, 0, rlo));
#pragma unroll
            for (int r = 0; r < QR; ++r) poly[pw + qf_pad(qf_rpart(r, lo))] = hi32(v[r]);
            if (rlo > 6) lds_sync();
            else lds_wave_order();
#pragma unroll
            for (int r = 0; r < QR; ++r) v[r] = with_hi(v[r], poly[pr + qf_pad(qf_rpart(r, rlo))]);
            lo = rlo;
        }
#pragma unroll
        for (int s = clo; s < chi; ++s) {
            const int b = s - rlo, bit = 1 << b;
#pragma unroll
            for (int r = 0; r < QR; ++r) {
                if (r & bit) continue;
                const int k = r & (bit - 1);
                if (s < 2 && k == 0) {   // power 1, values below 2q
                    const uint32_t x = hi32(v[r]), y = hi32(v[r | bit]);
                    v[r] = with_hi(v[r], x + y);
                    v[r | bit] = with_hi(v[r | bit], x - y + (s + 1) * q);
                } else {
                    if (MODE == NTT_LAZY) v[r] = with_hi(v[r], min(hi32(v[r]), hi32(v[r]) - 2 * q));
                    mont_bfly(v[r], v[r | bit], tw[bit - 1 + k], q, qn);
                }
            }
        }
    }
}

// Lazy Gentleman-Sande butterfly: (x, y) -> (x + y, (x - y) w), inputs and
// outputs in [0, 2q) for q < 2^30 (x - y + 2q < 4q fits 32 bits; Shoup's
// product without its correction lies in [0, 2q)).
__device__ __forceinline__ void qf_gs_bfly(uint32_t &x, uint32_t &y, uint32_t w, uint32_t ws, uint32_t q,
                                           uint32_t q2) {
    const uint32_t sum = x + y, d = x - y + q2;
    x = min(sum, sum - q2);
    y = d * w - __umulhi(d, ws) * q;
}

// Inverse transform (without the 1/N scale) of one polynomial held by N/16
// threads, stages ascending in chunks of four bits.  On entry register r of
// thread t holds position 16t + r of the bit-reversed arrangement (point
// bitrev(16t + r)); on return it holds N times coefficient
// qf_elem(t, r, LOGN - 4).  tw are the inverse twiddles (psi^-1 powers at
// bit-reversed indices) with companions at tws.  WIDE (q >= 2^30):
// canonical butterflies, outputs in [0, q); otherwise lazy, [0, 2q) from
// inputs in [0, 2q).  poly: LDS of N + N/16 words, of which since the last
// barrier a wave has read only its own 1024 elements' part.
template <int LOGN, bool WIDE>
__device__ __forceinline__ void intt_reg_block(uint32_t (&v)[QR], uint32_t t, uint32_t *poly,
                                               const uint32_t *tw, const uint32_t *tws, uint32_t q) {
    constexpr uint32_t n = 1u << LOGN;
    uint32_t lo = 0;
#pragma unroll
    for (int clo = 0; clo < LOGN; clo += 4) {
        const int chi = clo + 4 < LOGN ? clo + 4 : LOGN;
        const uint32_t rlo = (uint32_t)(clo < LOGN - 4 ? clo : LOGN - 4);   // registers cover [rlo, rlo + 4)
        if (rlo != lo) {
            if (lo > 6) lds_sync();   // the other waves have read what this one overwrites
            else lds_wave_order();
            const uint32_t pw = qf_pad(qf_elem(t, 0, lo)), pr = qf_pad(qf_elem(t, 0, rlo));
#pragma unroll
            for (int r = 0; r < QR; ++r) poly[pw + qf_pad(qf_rpart(r, lo))] = v[r];
            if (rlo > 6) lds_sync();
            else lds_wave_order();
#pragma unroll
            for (int r = 0; r < QR; ++r) v[r] = poly[pr + qf_pad(qf_rpart(r, rlo))];
            lo = rlo;
        }
        const uint32_t eb = qf_elem(t, 0, lo);
#pragma unroll
        for (int x = clo; x < chi; ++x) {
            const uint32_t bit = 1u << (x - (int)lo), mgroups = n >> (x + 1);
            const uint32_t gb = mgroups + (eb >> (x + 1));
#pragma unroll
            for (int r = 0; r < QR; ++r) {
                if (r & bit) continue;
                const uint32_t gi = gb + (qf_rpart(r, lo) >> (x + 1));
                if (WIDE) {
                    const uint32_t u = v[r], w = v[r | bit];
                    v[r] = add_mod_w(u, w, q);
                    v[r | bit] = mul_shoup_w(sub_mod(u, w, q), tw[gi], tws[gi], q);
                } else {
                    qf_gs_bfly(v[r], v[r | bit], tw[gi], tws[gi], q, 2 * q);
                }
            }
        }
    }
}

}  // namespace pir
