// RowSel on the INT8 matrix cores from the VALU layout, so that a DB without
// digit planes serves batches at the rate of its stream.
//
// The arithmetic is that of rowsel_mfma.hip (four balanced signed digits per
// residue, sixteen digit products summed per weight class s = i + j in int32,
// exact binary64 recombination per output, a class flush every 2048 rows of k).
// The DB's digits are cut on the way: the layout [L][N/4][S][D0][W][4] keeps
// four points of a record in 16 bytes, so a thread that loads eight consecutive
// rows k of one column holds, per point, the eight words whose byte d are eight
// k of digit plane d; two instructions a word make balanced digits of them and
// a byte transpose (v_perm_b32) eight contiguous bytes per digit.
//
// A persistent block of eight waves takes one point group (four points), 64
// columns and 16 RT query rows.  Per 64 rows of k every thread loads eight
// 16-byte vectors (1 KiB runs), cuts them and writes the digit rows to LDS
// (64 KiB, two buffers, one barrier a chunk); wave w then multiplies point
// w % 4 with v_mfma_i32_16x16x64_i8: with 32 rows one 16-row half of them times
// all 64 columns, with 16 rows one half of the columns.  Its query digits come
// from memory already in operand order.  The next chunk's loads, the next
// unit's too, are in flight during the products.
//
// Bound by HBM: per 64 KiB of DB the LDS moves 224 KiB and the matrix cores
// work 2048 cycles, together less than the 5800 cycles the read takes.
// 8 GiB (512 x 512, N = 4096, two limbs; GEMM alone): 4 clients 1.46 ms, 8
// clients 1.52 ms, 16 clients 1.68 ms, as fast as the digit planes' kernels;
// 13 clients on 333 x 301 (N = 2048, three limbs) 0.63 ms, 2.77 ms on the
// vector ALUs.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "common.h"
#include "mfma.h"
#include "modarith.h"

namespace pir {

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr uint32_t XCH = 64;          // rows of k per chunk
constexpr uint32_t XSUPER = 32;       // chunks per int32 accumulation (2048 rows)
constexpr uint32_t XCOLS = 64;        // columns of a unit
constexpr int XWAVES = 8;
constexpr int XBUF = 4 * 4 * XCOLS * XCH;   // LDS bytes of one chunk: [point][digit][column][64 k]
static_assert(VALU_STRIP % XCOLS == 0, "a unit's columns lie in one DB strip");

__device__ __forceinline__ void xbarrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Eight rows k = 8 wv .. + 7 of a chunk for one column (lane) and four points,
// cut into digits, to LDS [point][digit][column][64 k]: the 16-byte piece c of
// column n sits at c ^ ((n >> 1) & 3) (fragment reads free of bank conflicts).
template <bool WIDE>
__device__ __forceinline__ void cut_rows(int8_t *buf, const uint4 (&raw)[8], uint32_t lane, uint32_t wv, uint32_t q) {
    int8_t *const to = buf + lane * XCH + ((wv / 2) ^ ((lane >> 1) & 3)) * 16 + (wv % 2) * 8;
    auto transpose4 = [](uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint32_t (&o)[4]) {
        const uint32_t a = __builtin_amdgcn_perm(w1, w0, 0x06020400u);   // w0.0 w1.0 w0.2 w1.2
        const uint32_t c = __builtin_amdgcn_perm(w1, w0, 0x07030501u);   // w0.1 w1.1 w0.3 w1.3
        const uint32_t e = __builtin_amdgcn_perm(w3, w2, 0x06020400u);
        const uint32_t f = __builtin_amdgcn_perm(w3, w2, 0x07030501u);
        o[0] = __builtin_amdgcn_perm(e, a, 0x05040100u);
        o[1] = __builtin_amdgcn_perm(f, c, 0x05040100u);
        o[2] = __builtin_amdgcn_perm(e, a, 0x07060302u);
        o[3] = __builtin_amdgcn_perm(f, c, 0x07060302u);
    };
#pragma unroll
    for (int pi = 0; pi < 4; ++pi) {
        uint32_t w[8], lo[4], hi[4];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t x = pi == 0 ? raw[i].x : pi == 1 ? raw[i].y : pi == 2 ? raw[i].z : raw[i].w;
            w[i] = WIDE ? split_digits_window(x, q) : split_digits(x);
        }
        transpose4(w[0], w[1], w[2], w[3], lo);
        transpose4(w[4], w[5], w[6], w[7], hi);
#pragma unroll
        for (int d = 0; d < 4; ++d)
            *reinterpret_cast<uint2 *>(to + (pi * 4 + d) * (XCOLS * XCH)) = make_uint2(lo[d], hi[d]);
    }
}

template <int RT, int MODE>
__global__ void __launch_bounds__(64 * XWAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
rowsel_mfma_valu_kernel(const MfmaJob J, const uint4 *__restrict__ db, uint32_t d0) {
    constexpr int NS = RT == 2 ? 4 : 2;   // 16-column sub-tiles of a wave
    __shared__ __attribute__((aligned(1024))) int8_t lds[2 * XBUF];
    const uint32_t tid = threadIdx.x, lane = tid % 64;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid / 64);
    const uint32_t pw = wv % 4, hw = wv / 4;            // the wave's point, and its half of the rows or columns
    const uint32_t nkc = J.nkc, d1 = J.d1, units = J.tiles;
    const uint64_t qplane = (uint64_t)J.mstride * XCH, qstride = nkc * qplane;
    const uint32_t per_xcd = gridDim.x / 8, xcd = blockIdx.x % 8, yi = blockIdx.x / 8;
    auto unit_of = [&](uint32_t i) { return (i * 8 + xcd) * per_xcd + yi; };
    if (unit_of(0) >= units) return;   // uniform over the block

    // units of one XCD are consecutive: the row blocks of a column block share
    // its DB lines in that L2, the column blocks of a group its query digits
    struct Unit {
        uint32_t gg, l, m0, n0;
    };
    auto decode = [&](uint32_t u) {
        Unit r;
        r.m0 = u % J.nblk_m * (16 * RT);
        u /= J.nblk_m;
        r.n0 = u % J.nblk_n * XCOLS;
        r.gg = u / J.nblk_n;
        r.l = r.gg / (J.N / 4);
        return r;
    };

    // ---- load cursor: chunk l_kc of unit lu.  Thread: column tid % 64, rows
    // 8 (tid / 64) .. + 7 of the chunk (rows past D0 meet zero query digits)
    uint32_t li = 0, l_kc = 0;
    Unit lu = decode(unit_of(0));
    bool l_more = true;
    const uint4 *l_col;
    const int8_t *l_q;
    uint32_t l_w;
    auto l_start = [&]() {
        const uint32_t strip = lu.n0 / VALU_STRIP, c0 = lu.n0 % VALU_STRIP;
        l_w = valu_strip_width(strip, d1);
        l_col = db + valu_strip_base(lu.gg, strip, d0, d1) + min(c0 + lane, l_w - 1);   // (columns past D1: not stored)
        const uint64_t p = 4ull * lu.gg + pw;
        l_q = J.qd + p * 4 * qstride + (lu.m0 + (RT == 2 ? hw * 16 : 0) + lane % 16) * XCH + (lane / 16) * 16;
    };
    uint4 raw[8];
    i32x4 qn[4];   // the wave's query digits of the chunk in raw
    auto issue = [&]() {
        if (!l_more) return;
        const uint32_t k0 = l_kc * XCH + 8 * wv;
#pragma unroll
        for (int i = 0; i < 8; ++i) raw[i] = ld_nt(l_col + (uint64_t)min(k0 + i, d0 - 1) * l_w);
#pragma unroll
        for (int d = 0; d < 4; ++d) qn[d] = *reinterpret_cast<const i32x4 *>(l_q + d * qstride + l_kc * qplane);
        if (++l_kc == nkc) {
            l_kc = 0;
            l_more = unit_of(++li) < units;
            if (l_more) {
                lu = decode(unit_of(li));
                l_start();
            }
        }
    };

    i32x4 acc[7][NS];
    auto zero_acc = [&]() {
#pragma unroll
        for (int c = 0; c < 7; ++c)
#pragma unroll
            for (int s = 0; s < NS; ++s) acc[c][s] = (i32x4){0, 0, 0, 0};
    };
    zero_acc();
    Unit cu = lu;
    // Recombination of the classes into the staging layout [point][rows][sstride]
    // (a later flush of the unit adds to what the earlier ones stored).  A DB
    // fragment is the first operand, so a lane holds four consecutive columns
    // of one query row.
    auto flush = [&](bool first) {
        const EpiQ mq = J.q[cu.l];
        const uint32_t m = cu.m0 + (RT == 2 ? hw * 16 : 0) + lane % 16;
        const uint32_t c0 = cu.n0 + (RT == 2 ? 0 : hw * 32) + 4 * (lane / 16);
        uint32_t *const row = J.out + ((4ull * cu.gg + pw) * J.mp + m) * J.sstride;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            uint32_t v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int gr[7];
#pragma unroll
                for (int c = 0; c < 7; ++c) gr[c] = acc[c][s][r];
                v[r] = combine_classes<MODE>(gr, mq);
            }
            if (m < J.mp && c0 + 16 * s < d1) {   // (staging rows are padded to four columns)
                uint4 *o = reinterpret_cast<uint4 *>(row + c0 + 16 * s);
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

    l_start();
    issue();
    uint32_t b = 0;
    for (uint32_t ci = 0; unit_of(ci) < units; ++ci) {
        cu = decode(unit_of(ci));
        for (uint32_t kc = 0; kc < nkc; ++kc) {
            int8_t *const buf = lds + b * XBUF;
            b ^= 1;
            cut_rows<MODE == RECOMB_WIDE>(buf, raw, lane, wv, J.q[cu.l].q);
            i32x4 a[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) a[d] = qn[d];
            issue();
            // one barrier a chunk: a wave is past the one before only when its
            // reads of the other buffer are done
            xbarrier();
            const int8_t *bb = buf + pw * 4 * (XCOLS * XCH) + ((RT == 2 ? 0 : hw * 32) + lane % 16) * XCH +
                               ((lane / 16) ^ ((lane >> 1) & 3)) * 16;
            i32x4 f[2][NS];
            auto read_b = [&](int j) {
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    f[j % 2][s] = *reinterpret_cast<const i32x4 *>(bb + j * (XCOLS * XCH) + s * 16 * XCH);
            };
            read_b(0);
            read_b(1);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int s = 0; s < NS; ++s)
                        acc[i + j][s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[j % 2][s], a[i], acc[i + j][s], 0, 0, 0);
                if (j + 2 < 4) read_b(j + 2);
            }
            if (kc + 1 == nkc || (kc + 1) % XSUPER == 0) flush(kc < XSUPER);
        }
    }
}

// The digit planes [L*N][4][Kp/64][D1][64] of a DB from its VALU layout: a block
// takes a point group, 64 columns and a 64-row chunk, 1 KiB runs in and 4 KiB
// runs out; HBM-bound, 1 GiB in 0.36 ms (6.0 TB/s both ways).  grid: groups * nblk_n * chunks.
template <bool WIDE>
__global__ void __launch_bounds__(64 * XWAVES)
planes_from_valu_kernel(const uint4 *__restrict__ db, int8_t *__restrict__ planes, uint32_t d0, uint32_t d1,
                        uint32_t G, uint32_t nkc, uint32_t c0, uint32_t nblk_n, uint32_t nchunk, uint4 qs) {
    __shared__ __attribute__((aligned(1024))) int8_t lds[XBUF];
    const uint32_t tid = threadIdx.x, lane = tid % 64;
    const uint32_t wv = __builtin_amdgcn_readfirstlane(tid / 64);
    uint32_t b = blockIdx.x;
    const uint32_t n0 = b % nblk_n * XCOLS;
    b /= nblk_n;
    const uint32_t chunk = c0 + b % nchunk, gg = b / nchunk, l = gg / G;
    const uint32_t strip = n0 / VALU_STRIP, w = valu_strip_width(strip, d1);
    const uint4 *col = db + valu_strip_base(gg, strip, d0, d1) + min(n0 % VALU_STRIP + lane, w - 1);
    const uint32_t k0 = chunk * XCH + 8 * wv;
    uint4 raw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) raw[i] = k0 + i < d0 ? ld_nt(col + (uint64_t)(k0 + i) * w) : make_uint4(0, 0, 0, 0);
    cut_rows<WIDE>(lds, raw, lane, wv, l == 0 ? qs.x : l == 1 ? qs.y : l == 2 ? qs.z : qs.w);
    xbarrier();
#pragma unroll
    for (int j = 0; j < XBUF / 16 / (64 * XWAVES); ++j) {
        const uint32_t e = tid + 64 * XWAVES * j, kq = e % 4, n = e / 4 % XCOLS, pd = e / (4 * XCOLS);
        if (n0 + n >= d1) continue;
        const uint4 x = *reinterpret_cast<const uint4 *>(lds + (pd * XCOLS + n) * XCH + (kq ^ ((n >> 1) & 3)) * 16);
        st_nt(reinterpret_cast<uint4 *>(planes + (((16ull * gg + pd) * nkc + chunk) * d1 + n0 + n) * XCH + kq * 16), x);
    }
}

int valu_cu_count() {
    static int cached = 0;
    if (!cached) {
        int dev = 0;
        PIR_HIP(hipGetDevice(&dev));
        PIR_HIP(hipDeviceGetAttribute(&cached, hipDeviceAttributeMultiprocessorCount, dev));
    }
    return cached;
}

}  // namespace

void launch_db_planes_from_valu(const pir_db &db, uint32_t row0, uint32_t nrows, hipStream_t st) {
    const auto &p = db.p;
    const uint32_t nkc = db.mfma.kp / XCH, c0 = row0 / XCH, nchunk = (row0 + nrows + XCH - 1) / XCH - c0;
    const uint32_t nblk_n = (p.d1 + XCOLS - 1) / XCOLS;
    const uint64_t blocks = (uint64_t)p.nprimes * (p.n / 4) * nblk_n * nchunk;
    if (row0 % XCH || ((row0 + nrows) % XCH && row0 + nrows != p.d0) || blocks >= (1ull << 31))
        PIR_FAIL(PIR_EINVAL, "rows [%u, %u) are no whole chunks", row0, row0 + nrows);
    const uint4 qs = make_uint4(p.q[0], p.q[1], p.q[2], p.q[3]);
    auto go = [&](auto kern) {
        kern<<<(uint32_t)blocks, 64 * XWAVES, 0, st>>>(reinterpret_cast<const uint4 *>(db.valu.data), db.mfma.data, p.d0,
                                                      p.d1, p.n / 4, nkc, c0, nblk_n, nchunk, qs);
    };
    if (db.wide) go(&planes_from_valu_kernel<true>);
    else go(&planes_from_valu_kernel<false>);
    PIR_LAUNCH_CHECK();
}

void launch_rowsel_mfma_valu(const pir_db &db, const uint32_t *q, uint32_t B, uint32_t *out, hipStream_t st) {
    // scratch: query digit planes [P][4][Kp/64][rows][64], then the output
    // staging [P][2B][sstride]
    const uint32_t m_rows = 2 * B, rt = m_rows <= 16 ? 1 : 2, bm = 16 * rt;
    const uint32_t mstride = (m_rows + bm - 1) / bm * bm, kp = (db.p.d0 + 63) / 64 * 64;
    const size_t qbytes = ((size_t)db.slots() * 4 * mstride * kp + 255) / 256 * 256;
    const size_t sbytes = (size_t)db.slots() * m_rows * staging_stride(db.p.d1) * 4;
    StreamScratch buf(qbytes + sbytes, st);
    int8_t *qd = buf.as<int8_t>();
    launch_query_digits_rows(db, q, m_rows, qd, mstride, 0, st);
    MfmaJob job = make_mfma_job(db, qd, reinterpret_cast<uint32_t *>(qd + qbytes), B, 0, 2);
    job.nkc = kp / 64;
    job.mp = m_rows;
    job.mstride = mstride;
    job.nblk_m = mstride / bm;
    job.nblk_n = (db.p.d1 + XCOLS - 1) / XCOLS;
    const uint64_t units = (uint64_t)job.groups * job.nblk_m * job.nblk_n;
    if (units >= (1ull << 31)) PIR_FAIL(PIR_EINVAL, "too many work units");
    job.tiles = (uint32_t)units;
    const uint32_t grid = 8 * (uint32_t)std::max(1, valu_cu_count() / 8);
    {
        KernelTimer::Scope timed(st);
        auto go = [&](auto r, auto mode) {
            rowsel_mfma_valu_kernel<decltype(r)::value, decltype(mode)::value><<<grid, 64 * XWAVES, 0, st>>>(
                job, reinterpret_cast<const uint4 *>(db.valu.data), db.p.d0);
        };
        auto go_mode = [&](auto r) {
            switch (job.split) {
                case RECOMB_DIRECT: go(r, std::integral_constant<int, RECOMB_DIRECT>{}); break;
                case RECOMB_SPLIT: go(r, std::integral_constant<int, RECOMB_SPLIT>{}); break;
                default: go(r, std::integral_constant<int, RECOMB_WIDE>{}); break;
            }
        };
        if (rt == 1) go_mode(std::integral_constant<int, 1>{});
        else go_mode(std::integral_constant<int, 2>{});
        PIR_LAUNCH_CHECK();
    }
    launch_out_transpose(job.out, out, m_rows, m_rows, db.p.d1, (uint32_t)db.slots(), st);
}

}  // namespace pir
