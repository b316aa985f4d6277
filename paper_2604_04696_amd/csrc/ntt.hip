// Negacyclic NTT of arrays of polynomials, and the VALU layout of the DB.
//
// The transform turns coefficient-domain DB records into the NTT domain at
// load time (sec. 2.2 / sec. 2.4.1: records are kept NTT'd so RowSel is
// point-wise), takes a coefficient-domain query (the form query expansion
// leaves it in, sec. 2.2) there before RowSel, and serves clients and tests as
// the helper transform.  Convention: ahat_i = a(psi^(2i+1)), natural order.
//
// Cooley-Tukey butterflies with psi powers in bit-reversed order (forward,
// natural in -> bit-reversed positions) and Gentleman-Sande with inverse
// powers (inverse), the merged negacyclic formulation of Longa and Naehrig
// (CANS 2016).  All users hand over arrays of records of L polynomials, limb l
// of a record mod q_l, so one launch transforms every limb:
//   N >= 256  register-blocked (nttreg.h): N/16 threads hold 16 values each,
//             up to four butterfly stages per LDS exchange;
//   N < 256   one LDS stage per barrier, eight polynomials per block.
// The register-blocked form is bound by VALU issue (seven instructions per
// butterfly) with the memory traffic, one read and one write, close behind.
// On 1 GiB (65536 polynomials, N = 4096) it takes 0.45-0.47 ms; with Shoup's
// butterflies and barriers at every exchange 0.49-0.50 ms; one LDS stage per
// barrier, one launch per limb, 2.04 ms.
//
// Writing the MFMA path's digit planes straight from the transform (8 bytes of
// each 64-byte plane row per block) was measured and is not used: those
// scattered stores ran at a few hundred GB/s (7.9 ms for the 2 GiB query of 64
// clients).  One pass cannot write whole plane rows: a row needs the same
// point of all the 64 k of a chunk, i.e. 64 full polynomials (1 MiB at
// N = 4096) in one block.
#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <vector>

#include "common.h"
#include "modarith.h"
#include "nttreg.h"

namespace pir {

// ------------------------------------------------------------- host tables
uint32_t pow_mod(uint64_t a, uint64_t e, uint32_t q) {
    uint64_t r = 1 % q;
    a %= q;
    while (e) {
        if (e & 1) r = r * a % q;
        a = a * a % q;
        e >>= 1;
    }
    return (uint32_t)r;
}

static uint32_t smallest_generator(uint32_t q) {
    std::vector<uint32_t> f;
    uint32_t r = q - 1;
    for (uint32_t d = 2; (uint64_t)d * d <= r; ++d)
        if (r % d == 0) {
            f.push_back(d);
            while (r % d == 0) r /= d;
        }
    if (r > 1) f.push_back(r);
    for (uint32_t g = 2; g < q; ++g) {
        bool ok = true;
        for (uint32_t p : f)
            if (pow_mod(g, (q - 1) / p, q) == 1) { ok = false; break; }
        if (ok) return g;
    }
    PIR_FAIL(PIR_EINVAL, "no generator found for %u", q);
}

static uint32_t bitrev(uint32_t x, uint32_t logn) {
    uint32_t r = 0;
    for (uint32_t i = 0; i < logn; ++i) { r = (r << 1) | (x & 1); x >>= 1; }
    return r;
}

static uint32_t shoup(uint32_t w, uint32_t q) {
    return (uint32_t)(((uint64_t)w << 32) / q);
}

const NttTables &ntt_tables(uint32_t q, uint32_t n) {
    static std::mutex mu;
    static std::map<std::tuple<int, uint32_t, uint32_t>, NttTables> cache;
    int dev = 0;
    PIR_HIP(hipGetDevice(&dev));
    std::lock_guard<std::mutex> lock(mu);
    auto key = std::make_tuple(dev, q, n);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;

    uint32_t logn = 0;
    while ((1u << logn) < n) ++logn;
    uint32_t g = smallest_generator(q);
    uint32_t psi = pow_mod(g, (q - 1) / (2ull * n), q);
    uint32_t psi_inv = pow_mod(psi, q - 2, q);
    if (pow_mod(psi, n, q) != q - 1)
        PIR_FAIL(PIR_EINVAL, "psi is not a primitive 2N-th root mod %u", q);
    std::vector<uint32_t> fwd(6 * n), inv(4 * n);
    for (uint32_t k = 0; k < n; ++k) {
        uint32_t e = bitrev(k, logn);
        fwd[k] = pow_mod(psi, e, q);
        fwd[n + k] = shoup(fwd[k], q);
        fwd[2 * n + k] = (uint32_t)(((uint64_t)fwd[k] << 32) % q);
        inv[k] = pow_mod(psi_inv, e, q);
        inv[n + k] = shoup(inv[k], q);
    }
    for (uint32_t s = 0; (1u << s) < n; ++s) {
        const uint64_t w = pow_mod(psi_inv, 2ull * (n >> (s + 1)), q);
        uint64_t x = (1ull << 32) % q;
        for (uint32_t k = 0; k < 1u << s; ++k, x = x * w % q) inv[2 * n + (1u << s) + k] = (uint32_t)x;
    }
    uint64_t y = (1ull << 32) % q;
    for (uint32_t i = 0; i < n; ++i, y = y * psi_inv % q) inv[3 * n + i] = (uint32_t)y;
    for (uint32_t k = 0; k < n; ++k) {
        // the slot of tw_slot: group k is of stage x = logn - 1 - floor(log2 k)
        uint32_t at = k;
        const uint32_t T = n / 16;
        if (n >= 256 && k >= T) {
            uint32_t base = T, sh = 0;
            while (2 * base <= k) base *= 2, ++sh;
            at = base + ((k - base) & ((1u << sh) - 1)) * T + ((k - base) >> sh);
        }
        for (uint32_t part = 0; part < 3; ++part) fwd[(3 + part) * n + at] = fwd[part * n + k];
    }
    NttTables t;
    t.q = q;
    t.n = n;
    t.fwd = static_cast<uint32_t *>(dev_alloc(sizeof(uint32_t) * 6 * n));
    t.inv = static_cast<uint32_t *>(dev_alloc(sizeof(uint32_t) * 4 * n));
    PIR_HIP(hipMemcpy(t.fwd, fwd.data(), sizeof(uint32_t) * 6 * n, hipMemcpyHostToDevice));
    PIR_HIP(hipMemcpy(t.inv, inv.data(), sizeof(uint32_t) * 4 * n, hipMemcpyHostToDevice));
    t.n_inv = pow_mod(n, q - 2, q);
    t.n_inv_shoup = shoup(t.n_inv, q);
    uint32_t qi = q;   // Newton's iteration for q^-1 mod 2^32 (q q = 1 mod 8 for odd q)
    for (int i = 0; i < 4; ++i) qi *= 2 - q * qi;
    t.qn = 0u - qi;
    return cache.emplace(key, t).first->second;
}

// ------------------------------------------------------------------ kernels
struct NttPrimes {
    const uint32_t *tw[PIR_MAX_PRIMES];   // twiddles of the direction: [n] powers, [n] Shoup companions, forward also [n] Montgomery forms
    uint32_t q[PIR_MAX_PRIMES];
    uint32_t r1[PIR_MAX_PRIMES];          // floor(2^32 / q): Shoup companion of 1
    uint32_t ninv[PIR_MAX_PRIMES], ninv_s[PIR_MAX_PRIMES];
    uint32_t qn[PIR_MAX_PRIMES];          // -q^-1 mod 2^32
};

// Polynomials of a block: block b takes limb b % L of records
// (b / L) * PPB .. + PPB - 1 (ppb for small rings), so one block has one prime.
// (in may equal out: a block reads its polynomials whole before it writes.)

// Small rings (N < 256).  WIDE: some q >= 2^30, sums and Shoup products kept
// in 64 bits (modarith.h).  Up to NTS_PPB polynomials a block, fewer where that
// leaves fewer than NTS_BLOCKS blocks a limb: a waited-for call with 256
// polynomials of N = 128 takes 17.9 us with one each and 19.8 with eight.
constexpr uint32_t NTS_PPB = 8, NTS_THREADS = 256, NTS_MAX_N = 128, NTS_BLOCKS = 512;

template <bool INV, bool WIDE>
__global__ void __launch_bounds__(NTS_THREADS)
ntt_small_kernel(const uint32_t *in, uint32_t *out, uint32_t records, uint32_t L, uint32_t n, uint32_t logn,
                 uint32_t ppb, NttPrimes pr) {
    __shared__ uint32_t s[NTS_PPB * NTS_MAX_N];
    const uint32_t tid = threadIdx.x, l = blockIdx.x % L, r0 = blockIdx.x / L * ppb;
    const uint32_t polys = min(ppb, records - r0);
    const uint32_t q = pr.q[l], ninv = pr.ninv[l], ninv_s = pr.ninv_s[l];
    const uint32_t *tw = pr.tw[l], *tws = tw + n;
    auto addm = [&](uint32_t a, uint32_t b) { return WIDE ? add_mod_w(a, b, q) : add_mod(a, b, q); };
    auto mulm = [&](uint32_t a, uint32_t w, uint32_t ws) {
        return WIDE ? mul_shoup_w(a, w, ws, q) : mul_shoup(a, w, ws, q);
    };
    auto at = [&](uint32_t e) { return ((uint64_t)(r0 + (e >> logn)) * L + l) * n + (e & (n - 1)); };
    auto rev = [&](uint32_t e) { return (e >> logn << logn) | (__brev(e & (n - 1)) >> (32 - logn)); };

    for (uint32_t e = tid; e < polys * n; e += NTS_THREADS) {
        const uint32_t v = in[at(e)];
        s[INV ? rev(e) : e] = v >= q ? v % q : v;
    }
    __syncthreads();
    const uint32_t half = n >> 1;
    for (uint32_t st = 0; st < logn; ++st) {
        const uint32_t lt = INV ? st : logn - 1 - st, m = half >> lt, d = 1u << lt;
        for (uint32_t e = tid; e < polys * half; e += NTS_THREADS) {
            const uint32_t b = e & (half - 1), i = b >> lt;
            const uint32_t j = (e >> (logn - 1) << logn) + (i << (lt + 1)) + (b & (d - 1));
            const uint32_t u = s[j], v = s[j + d], w = tw[m + i], ws = tws[m + i];
            if (INV) {
                s[j] = addm(u, v);
                s[j + d] = mulm(sub_mod(u, v, q), w, ws);
            } else {
                const uint32_t t = mulm(v, w, ws);
                s[j] = addm(u, t);
                s[j + d] = sub_mod(u, t, q);
            }
        }
        __syncthreads();
    }
    for (uint32_t e = tid; e < polys * n; e += NTS_THREADS)
        out[at(e)] = INV ? mulm(s[e], ninv, ninv_s) : s[rev(e)];
}

// Register-blocked form (N >= 256): 256 threads per block up to N = 4096 (one
// polynomial there, several below), N/16 above.  Small blocks leave up to
// eight on a CU, so one block's loads and stores run under the others'
// butterflies.
template <int LOGN>
struct NttRegShape {
    static constexpr uint32_t n = 1u << LOGN, T = n / QR;
    static constexpr uint32_t PPB = T < 256 ? 256 / T : 1, THREADS = PPB * T;
};

template <int LOGN, bool INV, bool WIDE>
__global__ void __launch_bounds__(NttRegShape<LOGN>::THREADS)
ntt_reg_kernel(const uint32_t *in, uint32_t *out, uint32_t records, uint32_t L, NttPrimes pr) {
    using S = NttRegShape<LOGN>;
    constexpr uint32_t n = S::n, T = S::T;
    __shared__ uint32_t s[S::PPB * (n + n / 16)];
    const uint32_t t = threadIdx.x % T, pi = threadIdx.x / T;
    const uint32_t l = blockIdx.x % L, rec = blockIdx.x / L * S::PPB + pi;
    const bool live = S::PPB == 1 || rec < records;   // uniform per polynomial
    const uint32_t q = pr.q[l], r1 = pr.r1[l];
    const uint32_t *tw = pr.tw[l], *tws = tw + n;
    uint32_t *poly = s + pi * (n + n / 16);
    const uint64_t off = ((uint64_t)rec * L + l) * n;

    // any 32-bit value: x - floor(x * floor(2^32/q) / 2^32) * q is x mod q or
    // x mod q + q, in [0, 2q) as the lazy butterflies allow (for q >= 2^30,
    // canonical, with 64-bit intermediates).  The forward transform's first
    // stage pairs registers r and r + 8, and only its first operands need the
    // reduction: the second ones go into the butterfly's product, which takes
    // any 32-bit value.
    uint32_t v[QR];
#pragma unroll
    for (int r = 0; r < QR; ++r) {
        const uint32_t x = live ? __builtin_nontemporal_load(in + off + t + r * T) : 0u;
        if (WIDE) {
            const uint64_t y = (uint64_t)x - (uint64_t)__umulhi(x, r1) * q;
            v[r] = (uint32_t)(y >= q ? y - q : y);
        } else {
            v[r] = !INV && (r & 8) ? x : x - __umulhi(x, r1) * q;
        }
    }
    if constexpr (INV) {
        // point j goes to position bitrev(j) (t < T = 2^(LOGN-4): t and r T are
        // disjoint bit fields, see qf_rpart)
#pragma unroll
        for (int r = 0; r < QR; ++r)
            poly[qf_pad(__brev(t) >> (32 - LOGN)) + qf_pad(__brev((uint32_t)r * T) >> (32 - LOGN))] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < QR; ++r) v[r] = poly[qf_pad(t * QR) + r];
        intt_reg_block<LOGN, WIDE>(v, t, poly, tw, tws, q);
        const uint32_t ni = pr.ninv[l], nis = pr.ninv_s[l];
#pragma unroll
        for (int r = 0; r < QR; ++r)
            if (live) out[off + t + r * T] = WIDE ? mul_shoup_w(v[r], ni, nis, q) : mul_shoup(v[r], ni, nis, q);
    } else {
        constexpr int MODE = WIDE ? NTT_WIDE : NTT_LAZY;
        NttVal<MODE> x[QR];
#pragma unroll
        for (int r = 0; r < QR; ++r) x[r] = 0, ntt_set(x[r], v[r]);
        const TwGlobal src{WIDE ? tw : tw + 2 * n, tws};
        uint2 w0[QR];
        tw_first<LOGN>(w0, src);
        ntt_reg_block<LOGN, MODE>(x, t, poly, w0, src, q, pr.qn[l], [] {});
        // element 16t + r holds point bitrev(16t + r): natural order through
        // LDS, then coalesced stores
        lds_sync();
        const uint32_t pb = qf_pad(__brev(t * QR) >> (32 - LOGN));
#pragma unroll
        for (int r = 0; r < QR; ++r)
            poly[pb + qf_pad(__brev((uint32_t)r) >> (32 - LOGN))] = WIDE ? ntt_get(x[r]) : qf_reduce4(ntt_get(x[r]), q, 2 * q);
        lds_sync();
#pragma unroll
        for (int r = 0; r < QR; ++r)
            if (live) out[off + t + r * T] = poly[qf_pad(t) + qf_pad(r * T)];
    }
}

void launch_ntt(const uint32_t *in, uint32_t *out, uint64_t records, uint32_t n, uint32_t L, const uint32_t *q,
                bool inverse, hipStream_t st) {
    if (records == 0) return;
    uint32_t logn = 0;
    while ((1u << logn) < n) ++logn;
    NttPrimes pr{};
    bool wide = false;
    for (uint32_t l = 0; l < L; ++l) {
        const NttTables &t = ntt_tables(q[l], n);
        pr.tw[l] = inverse ? t.inv : t.fwd;
        pr.q[l] = q[l];
        pr.r1[l] = (uint32_t)((1ull << 32) / q[l]);
        pr.ninv[l] = t.n_inv;
        pr.ninv_s[l] = t.n_inv_shoup;
        pr.qn[l] = t.qn;
        wide = wide || q[l] >= WIDE_Q;
    }
    // a launch holds fewer than 2^32 threads (N/16 a polynomial, for small rings 32)
    const uint64_t most = (1ull << 31) / ((uint64_t)L * std::max(n / QR, 32u));
    for (uint64_t r0 = 0; r0 < records; r0 += most) {
        const uint32_t nr = (uint32_t)std::min(records - r0, most);
        const uint32_t *src = in + r0 * L * n;
        uint32_t *dst = out + r0 * L * n;
        auto go = [&](auto inv, auto w) {
            constexpr bool I = decltype(inv)::value, W = decltype(w)::value;
            auto reg = [&](auto lg) {
                using S = NttRegShape<decltype(lg)::value>;
                ntt_reg_kernel<decltype(lg)::value, I, W>
                    <<<(nr + S::PPB - 1) / S::PPB * L, S::THREADS, 0, st>>>(src, dst, nr, L, pr);
            };
            switch (logn) {
                case 8: reg(std::integral_constant<int, 8>{}); break;
                case 9: reg(std::integral_constant<int, 9>{}); break;
                case 10: reg(std::integral_constant<int, 10>{}); break;
                case 11: reg(std::integral_constant<int, 11>{}); break;
                case 12: reg(std::integral_constant<int, 12>{}); break;
                case 13: reg(std::integral_constant<int, 13>{}); break;
                case 14: reg(std::integral_constant<int, 14>{}); break;
                default: {
                    const uint32_t ppb = std::min(NTS_PPB, std::max(1u, nr / NTS_BLOCKS));
                    ntt_small_kernel<I, W><<<(nr + ppb - 1) / ppb * L, NTS_THREADS, 0, st>>>(src, dst, nr, L, n, logn,
                                                                                            ppb, pr);
                }
            }
        };
        if (inverse) {
            if (wide) go(std::true_type{}, std::true_type{});
            else go(std::true_type{}, std::false_type{});
        } else {
            if (wide) go(std::false_type{}, std::true_type{});
            else go(std::false_type{}, std::false_type{});
        }
        PIR_LAUNCH_CHECK();
    }
}

// ------------------------------------------- transform into the VALU layout
// Coefficients [nrows][D1][L][N] -> the VALU layout, with no NTT-domain copy in
// between: a block transforms LB_C consecutive columns of one row and limb into
// LDS (N/16 threads each) and writes 64-byte runs (LB_C columns of a point
// group), whose other half the next block, on the same XCD, brings to the same
// L2 line (64 registers: two blocks on a CU).  1 GiB of coefficients takes
// 0.56 ms (as a transform and a layout
// pass, which move twice the bytes, 0.45 and 0.37 ms); two columns a block
// 0.80 ms, two after the other in blocks of 512 threads 0.57-0.60 ms,
// non-temporal stores 0.66 ms.
constexpr uint32_t LB_C = 4;
static_assert(VALU_STRIP % LB_C == 0, "a block's columns lie in one strip");

template <int LOGN>
struct NttLayoutShape {
    static constexpr uint32_t n = 1u << LOGN, T = n / QR;
    static constexpr uint32_t THREADS = LB_C * T;
    static constexpr uint32_t PW = n + n / 16 + 1;   // (+ 1: the columns of a group in distinct banks)
};

template <int LOGN, bool WIDE>
__global__ void __launch_bounds__(NttLayoutShape<LOGN>::THREADS, 8)
ntt_layout_valu_kernel(const uint32_t *__restrict__ in, uint4 *__restrict__ dst, uint32_t row0, uint32_t d0,
                       uint32_t d1, uint32_t L, uint32_t nblk_n, NttPrimes pr) {
    using S = NttLayoutShape<LOGN>;
    constexpr uint32_t n = S::n, T = S::T;
    constexpr int MODE = WIDE ? NTT_WIDE : NTT_LAZY;
    extern __shared__ uint32_t s[];   // [LB_C][PW]
    const uint32_t t = threadIdx.x % T, pi = threadIdx.x / T;
    uint32_t b = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t n0 = b % nblk_n * LB_C;
    b /= nblk_n;
    const uint32_t l = b % L, row = b / L;
    const uint32_t q = pr.q[l], r1 = pr.r1[l];
    const TwGlobal src{WIDE ? pr.tw[l] : pr.tw[l] + 2 * n, pr.tw[l] + n};
    uint2 w0[QR];
    tw_first<LOGN>(w0, src);
    const uint32_t col = min(n0 + pi, d1 - 1);   // (columns past D1: not written)
    const uint32_t *from = in + (((uint64_t)row * d1 + col) * L + l) * n;
    uint32_t *poly = s + pi * S::PW;
    NttVal<MODE> v[QR];
    // any 32-bit value, as in ntt_reg_kernel
#pragma unroll
    for (int r = 0; r < QR; ++r) {
        const uint32_t x = __builtin_nontemporal_load(from + r * T + t);
        v[r] = 0;
        if (WIDE) {
            const uint64_t y = (uint64_t)x - (uint64_t)__umulhi(x, r1) * q;
            ntt_set(v[r], (uint32_t)(y >= q ? y - q : y));
        } else {
            ntt_set(v[r], r & 8 ? x : x - __umulhi(x, r1) * q);
        }
    }
    ntt_reg_block<LOGN, MODE>(v, t, poly, w0, src, q, pr.qn[l], [] {});
    lds_sync();
    const uint32_t pb = qf_pad(__brev(t * QR) >> (32 - LOGN));
#pragma unroll
    for (int r = 0; r < QR; ++r)
        poly[pb + qf_pad(__brev((uint32_t)r) >> (32 - LOGN))] =
            WIDE ? ntt_get(v[r]) : qf_reduce4(ntt_get(v[r]), q, 2 * q);
    lds_sync();
    const uint32_t strip = n0 / VALU_STRIP, w = valu_strip_width(strip, d1), c = threadIdx.x % LB_C;
    if (n0 + c >= d1) return;
    uint4 *to = dst + (uint64_t)(row0 + row) * w + (n0 + c) % VALU_STRIP;
    for (uint32_t g = threadIdx.x / LB_C; g < n / 4; g += S::THREADS / LB_C) {
        const uint32_t *x = s + c * S::PW + qf_pad(4 * g);
        to[valu_strip_base(l * (n / 4) + g, strip, d0, d1)] = make_uint4(x[0], x[1], x[2], x[3]);
    }
}

bool launch_ntt_layout_valu(const pir_db &db, const uint32_t *src, uint32_t row0, uint32_t nrows, hipStream_t st) {
    const auto &p = db.p;
    if (p.n < 256 || p.n > 4096) return false;
    const uint32_t nblk_n = (p.d1 + LB_C - 1) / LB_C, L = p.nprimes;
    if ((uint64_t)nblk_n * L * nrows >= (1ull << 31)) return false;
    NttPrimes pr{};
    bool wide = false;
    for (uint32_t l = 0; l < L; ++l) {
        const NttTables &t = ntt_tables(p.q[l], p.n);
        pr.tw[l] = t.fwd;
        pr.q[l] = p.q[l];
        pr.r1[l] = (uint32_t)((1ull << 32) / p.q[l]);
        pr.qn[l] = t.qn;
        wide = wide || p.q[l] >= WIDE_Q;
    }
    auto go = [&](auto lg, auto w) {
        constexpr int LG = decltype(lg)::value;
        using S = NttLayoutShape<LG>;
        auto kern = &ntt_layout_valu_kernel<LG, decltype(w)::value>;
        const size_t lds = LB_C * S::PW * sizeof(uint32_t);
        PIR_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
        kern<<<nblk_n * L * nrows, S::THREADS, lds, st>>>(src, reinterpret_cast<uint4 *>(db.valu.data), row0, p.d0, p.d1,
                                                         L, nblk_n, pr);
    };
    auto pick = [&](auto w) {
        switch (p.n) {
            case 256: go(std::integral_constant<int, 8>{}, w); break;
            case 512: go(std::integral_constant<int, 9>{}, w); break;
            case 1024: go(std::integral_constant<int, 10>{}, w); break;
            case 2048: go(std::integral_constant<int, 11>{}, w); break;
            default: go(std::integral_constant<int, 12>{}, w); break;
        }
    };
    if (wide) pick(std::true_type{});
    else pick(std::false_type{});
    PIR_LAUNCH_CHECK();
    return true;
}

// ------------------------------------------------------------ DB layouts
// NTT-domain source rows [nrows][D1][L*N/4] -> VALU layout [L*N/4][S][D0][W]
// (16-byte vectors of four points, 256-column strips, see DbLayoutValu).  The
// records of a strip, row after row, are one run of nrows * W vectors for each
// point group, so a tile takes LG groups of LC = 2048 / LG consecutive records,
// whatever the strip's width, through LDS: with LG = 32 512-byte read runs and
// 1 KiB write runs.  HBM-bound: 1 GiB in 0.36 ms (5.9 TB/s read and written);
// one vector per thread straight from the source, whose lanes read 16 bytes each
// from as many records, took 1.24 ms.  (Tiles of 64 columns of a single row are
// mostly empty where D1 is small: 16384 x 1 records of 32 KiB 2.12 ms, these
// 0.19.)  Non-temporal both ways: 128 MiB that no cache holds 49 us, with plain
// loads and stores 74 (42 against 48 where the same 128 MiB are loaded over and
// over).  The blocks walk the tiles: a launch holds fewer than 2^32 threads.
constexpr uint32_t LV_TILE = 2048, LV_THREADS = 256, LV_BLOCKS = 1u << 20;

template <uint32_t LG>
__global__ void __launch_bounds__(LV_THREADS)
db_layout_valu_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, uint32_t row0, uint32_t nrows,
                      uint32_t d0, uint32_t d1, uint32_t GG, uint32_t nblk_g, uint32_t per_strip, uint64_t tiles) {
    constexpr uint32_t LC = LV_TILE / LG, STEP = LV_THREADS / LG;   // (records between a thread's loads)
    static_assert(LC * LG == LV_TILE && STEP * LG == LV_THREADS, "a tile divides among the threads");
    __shared__ uint4 tile[LG][LC + 1];
    const uint32_t tid = threadIdx.x;
    for (uint64_t b = blockIdx.x; b < tiles; b += gridDim.x) {
        const uint32_t g0 = (uint32_t)(b % nblk_g) * LG, eb = (uint32_t)(b / nblk_g), strip = eb / per_strip;
        const uint32_t w = valu_strip_width(strip, d1), ne = nrows * w;   // records of the strip
        const uint32_t e0 = (eb - strip * per_strip) * LC;
        uint32_t e = e0 + tid / LG, r = e / w, c = e % w;
        const uint32_t dr = STEP / w, dc = STEP % w;
        uint4 v[LV_TILE / LV_THREADS];
#pragma unroll
        for (uint32_t j = 0; j < LV_TILE / LV_THREADS; ++j) {
            v[j] = g0 + tid % LG < GG && e < ne
                       ? ld_nt(src + ((uint64_t)r * d1 + strip * VALU_STRIP + c) * GG + g0 + tid % LG)
                       : make_uint4(0, 0, 0, 0);
            e += STEP, r += dr, c += dc;
            if (c >= w) c -= w, ++r;
        }
#pragma unroll
        for (uint32_t j = 0; j < LV_TILE / LV_THREADS; ++j) tile[tid % LG][j * STEP + tid / LG] = v[j];
        __syncthreads();
#pragma unroll
        for (uint32_t j = 0; j < LV_TILE / LV_THREADS; ++j) {
            const uint32_t f = j * LV_THREADS + tid, ci = f % LC, gi = f / LC;
            if (g0 + gi < GG && e0 + ci < ne)
                st_nt(dst + valu_strip_base(g0 + gi, strip, d0, d1) + (uint64_t)row0 * w + e0 + ci, tile[gi][ci]);
        }
        __syncthreads();
    }
}

void launch_db_layout_valu(const pir_db &db, const uint32_t *ntt_src, uint32_t row0,
                           uint32_t nrows, hipStream_t st) {
    const auto &p = db.p;
    if (!nrows) return;
    const uint32_t GG = p.nprimes * (p.n / 4);
    auto go = [&](auto lg) {
        constexpr uint32_t LG = decltype(lg)::value, LC = LV_TILE / LG;
        const uint32_t nblk_g = (GG + LG - 1) / LG, full = p.d1 / VALU_STRIP, rest = p.d1 % VALU_STRIP;
        const uint32_t per_strip = (nrows * VALU_STRIP + LC - 1) / LC;   // (nrows <= 65536)
        const uint64_t tiles = (uint64_t)nblk_g * ((uint64_t)full * per_strip + (nrows * rest + LC - 1) / LC);
        db_layout_valu_kernel<LG><<<(uint32_t)std::min<uint64_t>(tiles, LV_BLOCKS), LV_THREADS, 0, st>>>(
            reinterpret_cast<const uint4 *>(ntt_src), reinterpret_cast<uint4 *>(db.valu.data), row0, nrows, p.d0, p.d1,
            GG, nblk_g, per_strip, tiles);
    };
    // rings with fewer groups take tiles with fewer, and more records
    if (GG >= 32) go(std::integral_constant<uint32_t, 32>{});
    else if (GG >= 8) go(std::integral_constant<uint32_t, 8>{});
    else go(std::integral_constant<uint32_t, 2>{});
    PIR_LAUNCH_CHECK();
}

}  // namespace pir
