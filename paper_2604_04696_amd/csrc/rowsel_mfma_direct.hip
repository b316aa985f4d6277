// RowSel on the INT8 matrix cores for small batches (up to 32 query rows): the
// DB digit planes stream from HBM straight into the registers that the matrix
// instructions read, with no LDS copy and no barrier on their way.
//
// The arithmetic is that of rowsel_mfma.hip (four balanced signed digits per
// residue, sixteen digit products summed per weight class s = i + j in int32,
// exact binary64 recombination per output, a class flush every 2048 rows of k).
//
// A lane of v_mfma_i32_16x16x64_i8 supplies column l % 16 and the 16 bytes of
// k-group l / 16 of a 64-row chunk, and a column's chunk is 64 contiguous bytes
// of the digit plane: a fragment of 16 columns is one coalesced 1 KiB load,
// already in operand order.  A persistent block of eight waves takes a point
// (or a part of its columns) at a time: the query rows' digits for up to SEG
// chunks of k lie in one of two LDS buffers, the next point's are loaded into
// the other meanwhile, and the waves walk the columns 16 S at a time, each on
// its own, with NB chunks of the DB in registers (NB - 1 in flight, over the
// ends of tiles and points too).
//
// Bound by HBM: 16 matrix instructions per 4 KiB and 16 rows are a quarter of
// what the stream allows.  8 GiB (512 x 512, N = 4096, two limbs) take 1.30 ms
// for one client, the rate of a plain read; 8 clients 1.54 ms, of which 0.2 ms
// are the 0.25 GiB of results written beside it (as much when they leave in
// runs of 1 KiB, plain or non-temporal).  The tiled kernel, both operands
// through LDS in 32-row tiles, took 1.77 ms for either.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include "common.h"
#include "mfma.h"
#include "modarith.h"

namespace pir {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(3))) void lds_void;

constexpr uint32_t DKCH = 64;         // rows of k per chunk
constexpr uint32_t DSUPER = 32;       // chunks per int32 accumulation (2048 rows)

__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int N>
__device__ __forceinline__ void wait_vm() {
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int RT_, int S_, int W_, int NB_, int SEG_>
struct DShape {
    static constexpr int RT = RT_;     // 16-row sub-tiles of a unit (all of them in every wave)
    static constexpr int S = S_;       // 16-column sub-tiles per wave step
    static constexpr int W = W_;       // waves per block
    static constexpr int NB = NB_;     // DB chunk buffers per wave
    static constexpr int SEG = SEG_;   // chunks of k per LDS buffer of query digits (two buffers)
    static constexpr int ROWS = 16 * RT;
    static constexpr uint32_t RW = 16 * S * W;             // columns of a round (one step of every wave)
    static constexpr int CHUNK = 4 * ROWS * (int)DKCH;   // LDS bytes of one query chunk
    static_assert(4 * RT % W == 0 || W % (4 * RT) == 0, "query loads divide among the waves");
};

template <class D, int MODE>
__global__ void __launch_bounds__(64 * D::W) __attribute__((amdgpu_waves_per_eu(2, 4)))
rowsel_mfma_direct_kernel(const MfmaJob J) {
    constexpr int RT = D::RT, S = D::S, W = D::W, NB = D::NB, SEG = D::SEG, ROWS = D::ROWS;
    constexpr uint32_t RW = D::RW;   // columns of a round
    constexpr int AHEAD = 4 * S * (NB - 1);   // DB loads of a wave in flight beyond the chunk in use
    extern __shared__ __attribute__((aligned(1024))) int8_t qlds[];   // 2 x [chunk][digit][row][64]
    const uint32_t tid = threadIdx.x, lane = tid % 64;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid / 64);
    const uint32_t nkc = J.nkc, d1 = J.d1, units = J.tiles;
    const uint64_t qplane = (uint64_t)J.mstride * DKCH, dplane = (uint64_t)d1 * DKCH;
    const uint64_t qstride = nkc * qplane, dstride = nkc * dplane;   // one digit's planes
    // some segment is used for fewer chunks than a wave has DB buffers
    const bool drain = (nkc <= (uint32_t)SEG ? nkc : nkc % SEG ? nkc % SEG : (uint32_t)SEG) < (uint32_t)NB;
    const uint32_t seg_bytes = min((uint32_t)SEG, nkc) * D::CHUNK;
    // units of one XCD are consecutive: the column parts of a point share its
    // query planes in that L2
    const uint32_t per_xcd = gridDim.x / 8, xcd = blockIdx.x % 8, yi = blockIdx.x / 8;
    auto unit_of = [&](uint32_t i) { return (i * 8 + xcd) * per_xcd + yi; };
    if (unit_of(0) >= units) return;   // uniform over the block

    struct Unit {
        uint64_t p;                       // point l * N + j
        uint32_t pl, l, cb, rounds;   // staging point, prime, column part, wave steps of it
    };
    // column part cb of a point takes its rounds cb, cb + nblk_n, ... of RW columns
    const uint32_t nrounds = (d1 + RW - 1) / RW;
    auto decode = [&](uint32_t u) {
        Unit r;
        r.cb = u % J.nblk_n;
        r.pl = u / J.nblk_n;
        const uint32_t G = J.N / 4, gg = J.g_begin + r.pl / 4;
        r.l = gg / G;
        r.p = (uint64_t)r.l * J.N + 4 * (gg % G) + r.pl % 4;
        r.rounds = (nrounds - r.cb + J.nblk_n - 1) / J.nblk_n;
        return r;
    };
    auto round_col = [&](const Unit &t, uint32_t round) { return (t.cb + round * J.nblk_n) * RW; };

    // ---- DB cursor: chunk l_kc of round l_round of unit lu
    i32x4 buf[NB][4][S];
    uint32_t li = 0, l_round = 0, l_kc = 0;
    Unit lu = decode(unit_of(0));
    bool l_more = true;
    const int8_t *l_src[S];
    auto l_start = [&]() {
        const int8_t *base = J.dbd + lu.p * 4 * dstride + (lane / 16) * 16;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const uint32_t n = round_col(lu, l_round) + (wv * S + s) * 16 + lane % 16;
            l_src[s] = base + (uint64_t)min(n, d1 - 1) * DKCH;   // columns past D1 are never stored
        }
    };
    auto issue = [&](i32x4 (&b)[4][S]) {
        if (!l_more) return;
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int s = 0; s < S; ++s)
                b[d][s] = __builtin_nontemporal_load(reinterpret_cast<const i32x4 *>(l_src[s] + d * dstride));
        if (++l_kc == nkc) {
            l_kc = 0;
            if (++l_round == lu.rounds) {
                l_round = 0;
                l_more = unit_of(++li) < units;
                if (!l_more) return;
                lu = decode(unit_of(li));
            }
            l_start();
        } else {
#pragma unroll
            for (int s = 0; s < S; ++s) l_src[s] += dplane;
        }
    };

    // ---- query cursor: the segment after the one in use goes to the other
    // LDS buffer.  A load moves 16 rows of one digit and chunk (1 KiB); the
    // 16-byte piece c of row r sits at c ^ ((r >> 1) & 3) (fragment reads free
    // of bank conflicts), hence the lane's source offset.
    const uint32_t qlane = (lane / 4) * DKCH + ((lane % 4) ^ ((lane / 8) & 3)) * 16;
    uint32_t qi = 0, q_round = 0, q_c0 = 0, q_buf = 0;   // of the segment to load next
    Unit qu = lu;
    bool q_more = true;
    auto q_issue = [&]() {
        if (!q_more) return;
        const uint32_t count = min((uint32_t)SEG, nkc - q_c0);
        const int8_t *src = J.qd + qu.p * 4 * qstride + q_c0 * qplane + qlane;
        int8_t *dst = qlds + q_buf * seg_bytes;
        for (uint32_t v = wv; v < count * 4 * RT; v += W) {
            const uint32_t rb = v % RT, d = v / RT % 4, c = v / (4 * RT);
            __builtin_amdgcn_global_load_lds(src + d * qstride + c * qplane + rb * 1024, (lds_void *)(dst + v * 1024),
                                             16, 0, 0);
        }
        q_buf ^= 1;
        q_c0 += SEG;
        if (q_c0 >= nkc) {
            q_c0 = 0;
            // one segment serves every round when it holds all of k
            if (nkc <= (uint32_t)SEG || ++q_round == qu.rounds) {
                q_round = 0;
                q_more = unit_of(++qi) < units;
                if (q_more) qu = decode(unit_of(qi));
            }
        }
    };

    i32x4 acc[7][RT][S];
    auto zero_acc = [&]() {
#pragma unroll
        for (int c = 0; c < 7; ++c)
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int s = 0; s < S; ++s) acc[c][t][s] = (i32x4){0, 0, 0, 0};
    };
    zero_acc();
    // ---- compute cursor
    uint32_t ci = 0, round = 0, kc = 0, c_buf = 1, seg_left = 0, seg_at = 0;
    Unit cu = lu;
    // Recombination of the classes into the staging layout [point][rows][sstride]
    // (every SUPER chunks, and at the end of a round; a later flush adds to
    // what the earlier ones stored).  A DB fragment is the first operand, so a
    // lane holds four consecutive columns of one query row: one 16-byte store.
    auto flush = [&](bool first) {
        const EpiQ mq = J.q[cu.l];
        const uint32_t c0 = round_col(cu, round) + wv * S * 16 + 4 * (lane / 16);
        uint32_t *const pt = J.out + (uint64_t)cu.pl * J.mp * J.sstride;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const uint32_t m = t * 16 + lane % 16, n = c0 + s * 16;
                uint32_t v[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    int gr[7];
#pragma unroll
                    for (int c = 0; c < 7; ++c) gr[c] = acc[c][t][s][r];
                    v[r] = combine_classes<MODE>(gr, mq);
                }
                if (m < J.mp && n < d1) {   // (staging rows are padded to four columns)
                    uint4 *o = reinterpret_cast<uint4 *>(pt + (uint64_t)m * J.sstride + n);
                    if (!first) {
                        const uint4 was = *o;
                        auto add = [&](uint32_t x, uint32_t y) {
                            return MODE == RECOMB_WIDE ? add_mod_w(x, y, mq.q) : add_mod(x, y, mq.q);
                        };
                        v[0] = add(was.x, v[0]);
                        v[1] = add(was.y, v[1]);
                        v[2] = add(was.z, v[2]);
                        v[3] = add(was.w, v[3]);
                    }
                    *o = make_uint4(v[0], v[1], v[2], v[3]);
                }
                __builtin_amdgcn_sched_barrier(0);   // (the outputs one after the other: fewer registers)
            }
        zero_acc();
    };
    const uint32_t a_lane = (lane % 16) * DKCH + ((lane / 16) ^ ((lane >> 1) & 3)) * 16;
    // one chunk; returns whether it was the block's last
    auto step = [&](const i32x4 (&b)[4][S], bool start) {
        if (seg_left == 0) {
            // the next segment: this wave's loads of it are older than the DB
            // loads in flight (a segment is used for at least NB chunks, else
            // everything is waited for), then everybody's; after the
            // barrier the buffer of the segment before it is free
            if (start || drain) wait_vm<0>();
            else wait_vm<AHEAD>();
            lds_barrier();
            q_issue();
            asm volatile("" ::: "memory");
            c_buf ^= 1;
            seg_at = 0;
            seg_left = nkc <= (uint32_t)SEG ? nkc * cu.rounds : min((uint32_t)SEG, nkc - kc);
        }
        const int8_t *ab = qlds + c_buf * seg_bytes + seg_at * D::CHUNK + a_lane;
        i32x4 a[2][RT];
        auto read_a = [&](int i) {
#pragma unroll
            for (int t = 0; t < RT; ++t) a[i % 2][t] = *reinterpret_cast<const i32x4 *>(ab + (i * ROWS + t * 16) * DKCH);
        };
        read_a(0);
        read_a(1);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < RT; ++t)
#pragma unroll
                    for (int s = 0; s < S; ++s)
                        acc[i + j][t][s] =
                            __builtin_amdgcn_mfma_i32_16x16x64_i8(b[j][s], a[i % 2][t], acc[i + j][t][s], 0, 0, 0);
            if (i + 2 < 4) read_a(i + 2);
        }
        --seg_left;
        ++seg_at;
        ++kc;
        if (kc == nkc || kc % DSUPER == 0) flush(kc <= DSUPER);
        if (kc == nkc) {
            kc = 0;
            if (nkc <= (uint32_t)SEG) seg_at = 0;
            if (++round == cu.rounds) {
                round = 0;
                if (unit_of(++ci) >= units) return true;
                cu = decode(unit_of(ci));
            }
        }
        return false;
    };

    q_issue();
    asm volatile("" ::: "memory");
    l_start();
#pragma unroll
    for (int b = 0; b + 1 < NB; ++b) issue(buf[b]);
    bool start = true;
    for (;;) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            issue(buf[(b + NB - 1) % NB]);
            if (step(buf[b], start)) return;
            start = false;
        }
    }
}

int direct_cu_count() {
    static int cached = 0;
    if (!cached) {
        int dev = 0;
        PIR_HIP(hipGetDevice(&dev));
        PIR_HIP(hipDeviceGetAttribute(&cached, hipDeviceAttributeMultiprocessorCount, dev));
    }
    return cached;
}

}  // namespace

// Unit shapes by the rows of a call.  Up to 16 rows a wave takes 32 columns a
// step, unless rounds of 256 columns pad D1 by more than an eighth: then 16,
// with a third chunk in flight.  512 x 512, N = 4096, two limbs (GEMM alone):
// 16 rows 1.54 ms and 1.57 ms, 333 x 301, N = 2048, three limbs, 32 rows
// (16 columns) 0.62 ms; with a third buffer at 32 columns 1.55 ms.
static bool direct_narrow(uint32_t d1) { return (d1 + 255) / 256 * 256 > d1 + d1 / 8; }

// The kernel's rows for a call of `rows` query rows (0: another kernel's
// call).  Measured against the tiled kernel, GEMM alone, on the 512 x 512
// N = 4096 DB: 8 clients 1.54 ms against 1.77, 4 clients with 32-bit primes
// 1.47 against 1.79, 16 clients 1.73 against 1.79, and on ragged or small DBs
// the same or faster (1300 x 37, 15 clients 0.19 against 0.20 ms); at 64 rows
// the query-resident kernel is the faster one, 2.12 against 2.36.  With fewer than
// 64 columns half of a block's waves and more have none, and with more than one
// LDS segment of k the block waits for each: there 32 rows are the tiled
// kernel's, which takes four points a tile, where these give every CU one (16
// clients, N = 1024, us: 4096 x 16 479 and 459, 4096 x 48 538 and 493, 4096 x 64 567
// and 568, 4096 x 80 626 and 683, 640 x 32 96 and 85; in one segment 256 x 4 42 and 47;
// 4096 x 16 at N = 256, 128 tiles, 132 and 228).  16 rows are not (4 clients,
// 4096 x 48 at N = 1024 350 and 488).
constexpr uint32_t DSEG = 8;   // chunks of k per LDS segment, every shape

uint32_t direct_rows(uint32_t rows, uint32_t d1, uint32_t nkc, uint32_t groups) {
    if (const char *e = std::getenv("PIR_MFMA_KERNEL"))   // a kernel forced by name (tuning runs, tests)
        if (!std::strcmp(e, "qres") || !std::strcmp(e, "tile")) return 0;
    if (rows <= 16) return 16;
    return rows > 32 || (d1 < 64 && nkc > DSEG && groups >= (uint32_t)direct_cu_count()) ? 0 : 32;
}

void launch_mfma_direct(const MfmaJob &job0, hipStream_t st) {
    MfmaJob job = job0;
    if (!job.groups || !job.m_rows) return;
    auto go = [&](auto shape, auto mode) {
        using D = decltype(shape);
        constexpr int MODE = decltype(mode)::value;
        if (job.mp > (uint32_t)D::ROWS || (uint32_t)D::ROWS > job.mstride)
            PIR_FAIL(PIR_EINVAL, "query planes of %u rows hold no %d-row units", job.mstride, D::ROWS);
        const size_t lds = (size_t)2 * std::min<uint32_t>(job.nkc, D::SEG) * D::CHUNK;
        // persistent blocks, as many per CU as registers and LDS hold; a
        // point's columns are parted where there are few points
        const uint32_t per_cu = D::RT == 1 && D::S == 1 && lds <= 80 * 1024 ? 2u : 1u;
        const uint32_t grid = 8 * std::max(1u, (uint32_t)direct_cu_count() * per_cu / 8);
        const uint32_t rounds = (job.d1 + D::RW - 1) / D::RW, points = 4 * job.groups;
        job.nblk_n = 1;
        while (job.nblk_n < rounds && (uint64_t)points * job.nblk_n < 8 * grid) ++job.nblk_n;
        const uint64_t units = (uint64_t)points * job.nblk_n;
        if (units >= (1ull << 31)) PIR_FAIL(PIR_EINVAL, "too many work units");
        job.tiles = (uint32_t)units;
        auto kern = &rowsel_mfma_direct_kernel<D, MODE>;
        PIR_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
        kern<<<grid, 64 * D::W, lds, st>>>(job);
    };
    auto go_mode = [&](auto shape) {
        switch (job.split) {
            case RECOMB_DIRECT: go(shape, std::integral_constant<int, RECOMB_DIRECT>{}); break;
            case RECOMB_SPLIT: go(shape, std::integral_constant<int, RECOMB_SPLIT>{}); break;
            default: go(shape, std::integral_constant<int, RECOMB_WIDE>{}); break;
        }
    };
    if (job.mp > 16) go_mode(DShape<2, 1, 8, 3, DSEG>{});
    else if (direct_narrow(job.d1)) go_mode(DShape<1, 1, 8, 3, DSEG>{});
    else go_mode(DShape<1, 2, 8, 2, DSEG>{});
    PIR_LAUNCH_CHECK();
}

}  // namespace pir
