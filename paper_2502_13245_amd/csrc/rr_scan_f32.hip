// rr_scan_f32.hip -- dense float32 scan: a bfloat16 filter on the matrix
// cores in front of the exact FP64 decision.
//
// Every value is split into two bfloat16 parts, x = xh + xl + e with
// |e| <= 2^-18 |x|, and the products qh.xh + qh.xl + ql.xh accumulate in
// float32 (v_mfma_f32_32x32x16_bf16, three products a step).  A bound on the
// distance of that sum from q.x (slack, below) turns it into a test that no
// pair inside the radius can fail; the few pairs that pass are decided, and
// their distances computed, in FP64 from the float32 rows, chunk by chunk in
// the order of the graph search's kernels, so a scan and a search report the
// same bits.  Where many pairs pass (large radii, values far from the origin
// or of very different lengths) whole tiles are decided that way
// (k_split_dense).
//
// What bounds it: the float64 products would take 5.4 ms for 2,000 queries x
// 1M x 96 values at the 70 TFLOP/s that a large FP64 matrix product reaches
// on MI355X; three bfloat16 products are 0.9 ms at 1.27 PFLOP/s.  This kernel
// takes 1.42 ms (0.81 PFLOP/s of products).  The FP64 scan of rr_scan.hip took
// 30.4 ms (both operands read from memory at every step); it remains for data
// whose squares leave the float32 range.  Nearest distances (two passes): 2,000
// queries x 100K x 96 3.24 -> 0.27 ms, one query 74 -> 47 us, 100 queries x
// 100K x 200 468 -> 281 us.  Relative error of the FP64 results against a
// 64-bit reference: at most 1.1e-16 (differences), 1.2e-14 before (products).
//
// Layout: a workgroup of four waves holds 128 queries, 32 per wave, in
// registers (both parts; for rows of more than 128 values a step's part) and
// streams tiles of 64 base points: the tile's float32 rows are loaded one
// step ahead, split in registers and stored to LDS once for the four waves.
// Chunks of 16 bytes are stored at (chunk xor a function of the row), so the
// 16 lanes that read one chunk column of 16 rows fall on different banks.
// The test of a tile is one maximum over the 16 accumulators of a lane: they
// start at the query's threshold term, and the point's |x|^2 / 2 is constant
// along a lane.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "rr_scan.h"
#include "rr_search.h"

namespace rr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// SPLIT_MAX: the largest approximate q.x - |x|^2 / 2 of every query;
// SPLIT_RANGE: hits to the item arrays; SPLIT_MIN: the smallest distance of
// the pairs that pass
enum { SPLIT_MAX = 0, SPLIT_RANGE = 1, SPLIT_MIN = 2 };

constexpr int SPLIT_TILE = 64;   // base points per step
constexpr int SPLIT_Q = 128;     // queries per workgroup
constexpr int SPLIT_STAGE = 128; // staged candidates per wave
// A tile of 64 points and a wave's 32 queries with SPLIT_DENSE candidates (of
// 2,048 pairs) is left to k_split_dense, and so are the tiles that follow it
// with SPLIT_STAY.  That kernel takes 13 ps a pair of 96 values and 95 ps of 768
// (a tile 27 and 195 ns); a candidate decided by itself takes 60 to 145 ps and
// 650 ps, in a wave that its workgroup waits for.  200,000 x 96, 500 queries,
// a radius that 10% (20%) of the pairs lie in: 6.97 (12.3) ms from 384, 7.16
// (12.1) from 256, 7.8 (11.1) from 192, 7.9 (10.8) from 128; 50,000 x 768 with
// 20% 10.8, 9.1, 6.9 and 6.7.
constexpr int SPLIT_DENSE = 192;
constexpr int SPLIT_STAY = 128;

struct SplitArgs {
    ScanArgs sc;
    uint4 *dense;        // [dense_cap] runs of such tiles: 32-query block, first point, end
    unsigned long long *dense_cnt;
    int64_t dense_cap;   // 0: none are kept
    int32_t run_max;     // tiles of a run
    const uint16_t *qs;  // [nq][2][kpad] high and low parts of the queries
    const float *cinit;  // [nq] what the sums start from
    unsigned *best;      // [nq] SPLIT_MAX: ordered bits of the largest sum
    int64_t groups;      // workgroups
    int32_t kpad, cpl, g;
};

__device__ __forceinline__ unsigned flt_order(float f) {
    const unsigned b = __float_as_uint(f);
    return (b >> 31) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float flt_unorder(unsigned k) {
    return __uint_as_float((k >> 31) ? (k & 0x7fffffffu) : ~k);
}

// eight values as bfloat16: the rounded values and what they leave
__device__ __forceinline__ void split8(f32x8 x, uint4 &hi, uint4 &lo) {
    hi = __builtin_bit_cast(uint4, __builtin_convertvector(x, bf16x8));
    const uint32_t w[4] = {hi.x, hi.y, hi.z, hi.w};
    f32x8 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        r[2 * j] = x[2 * j] - __uint_as_float(w[j] << 16);
        r[2 * j + 1] = x[2 * j + 1] - __uint_as_float(w[j] & 0xffff0000u);
    }
    lo = __builtin_bit_cast(uint4, __builtin_convertvector(r, bf16x8));
}

// Split queries and their threshold terms, one wave per query.  With s the
// approximate sum of q.x and M the largest |x|, |s - q.x| is at most
// 3.1 2^-18 |q| M (the parts left out) plus (3 K + 16) 2^-22 times the
// magnitudes that the accumulation meets (K values a row; every addition and
// the comparison within 2^-22 of its operands), plus what underflows.
// Squared distance: d <= r  <=>  q.x - |x|^2 / 2 >= (|q|^2 - r) / 2; inner
// product: d <= r  <=>  q.x >= -r.  cinit is the negated right side plus the
// slack, rounded up.  A query that is not finite or too large to square in
// float32 gets zero parts and an infinite slack: every pair passes to the
// FP64 decision.
__global__ void k_split_prep(const uint8_t *qpad, const QThresh *qth, int64_t nq, int32_t row_bytes,
                             int32_t d, int32_t kpad, double maxnorm, int ip, uint16_t *qs, float *cinit,
                             float *slack_out, unsigned *best, unsigned long long *dense_cnt) {
    const int lane = threadIdx.x & 63;
    const int64_t w0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (w0 == 0 && lane == 0) *dense_cnt = 0ull;
    for (int64_t q = w0; q < nq; q += (int64_t)gridDim.x * (blockDim.x >> 6)) {
        const float *qr = reinterpret_cast<const float *>(qpad + q * row_bytes);
        double n2 = 0.0;
        for (int i = lane; i < d; i += 64) n2 = fma((double)qr[i], (double)qr[i], n2);
        for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
        const bool ok = n2 <= 1e34;
        const double qn = sqrt(n2), m = maxnorm * (1.0 + 1e-6);
        const double acc = (double)(3 * kpad + 16) * 0x1p-22;
        const double r = qth ? qth[q].r : 0.0;
        double slack = (3.2 * 0x1p-18 + acc) * qn * m + acc * 0.5 * (n2 + m * m + (qth ? fabs(r) : qn * m)) +
                       (qn + m) * (double)kpad * 0x1p-120 + 1e-30;
        if (!ok) slack = __builtin_huge_val();
        uint4 *hi = reinterpret_cast<uint4 *>(qs + (size_t)q * 2 * kpad), *lo = hi + kpad / 8;
        const int cols = row_bytes / 4;
        for (int c = lane; c < kpad / 8; c += 64) {
            f32x8 x = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (ok && c * 8 < cols) x = *reinterpret_cast<const f32x8 *>(qr + c * 8);
            uint4 h, l;
            split8(x, h, l);
            hi[c] = h;
            lo[c] = l;
        }
        if (lane == 0) {
            cinit[q] = ok ? __double2float_ru((ip ? r : 0.5 * (r - n2)) + slack) : __builtin_huge_valf();
            slack_out[q] = __double2float_ru(slack);
            best[q] = 0u; // below the ordered bits of every sum
        }
    }
}

// SPLIT_MIN's start: a pair can hold the query's smallest distance only if
// its sum comes within two slacks of the largest sum
__global__ void k_split_best(const unsigned *best, const float *slack, int64_t nq, float *cinit,
                             unsigned long long *nn_bits) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= nq) return;
    // (an infinite slack passes every pair, whatever the sums were)
    const double s = (double)slack[q];
    cinit[q] = s <= 1e38 ? __double2float_ru(2.0 * s - (double)flt_unorder(best[q])) : __builtin_huge_valf();
    nn_bits[q] = dbl_order(__builtin_huge_val());
}

// a wave's staged hits to the item arrays, with one cursor atomic, and one
// count per run of hits of a query
__device__ __forceinline__ void split_emit(const SplitArgs &a, const uint32_t *st_q, const uint32_t *st_id,
                                           const double *st_d, int n, int lane) {
    wave_sync();
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(a.sc.item_cursor, (unsigned long long)n);
    base = __shfl(base, 0);
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int i = i0 + lane;
        const int64_t pos = (int64_t)base + i;
        const bool in = i < n && pos < a.sc.item_cap; // (a prefix of the lanes)
        const uint32_t q = in ? st_q[i] : ~0u, before = __shfl_up(q, 1);
        if (in) {
            a.sc.item_key[pos] = ((unsigned long long)q << 32) | st_id[i];
            ((double *)a.sc.item_dist)[pos] = st_d[i];
        }
        const bool head = in && (lane == 0 || before != q);
        const unsigned long long hm = __ballot(head), im = __ballot(in); // (by every lane)
        const unsigned long long later = hm & ~((2ull << lane) - 1ull);
        const int end = later ? __ffsll((long long)later) - 1 : __popcll(im);
        if (head) atomicAdd(&a.sc.task_cnt[q], (unsigned long long)(end - lane));
    }
    if (lane == 0 && (int64_t)base + n > a.sc.item_cap) atomicOr(a.sc.overflow, 64ull);
    wave_sync();
}

// The staged pairs of one wave, decided in FP64: groups of g lanes read a
// pair's rows, each lane cpl chunks, summed as eval64 sums them.  Hits are
// compacted in place (a round's reads precede its writes, which land at or
// below its first entry) and appended to the item arrays (SPLIT_RANGE), or
// lower their query's minimum (SPLIT_MIN).
template <int MODE>
__device__ __forceinline__ void split_flush(const SplitArgs &a, uint32_t *st_q, uint32_t *st_id,
                                            double *st_d, int n, int lane) {
    wave_sync();
    const int g = a.g, cpl = a.cpl, gl = lane & (g - 1), per = 64 / g;
    const bool ip = a.sc.ix.metric == RR_IP;
    const size_t rb = a.sc.ix.row_bytes;
    int kept = 0; // (hits)
    for (int e0 = 0; e0 < n; e0 += per) {
        const int e = e0 + lane / g;
        const uint32_t q = st_q[min(e, n - 1)], id = st_id[min(e, n - 1)];
        const uint4 *x = reinterpret_cast<const uint4 *>(a.sc.ix.base + id * rb) + gl * cpl;
        const uint4 *y = reinterpret_cast<const uint4 *>(a.sc.qpad + q * rb) + gl * cpl;
        double s = 0.0;
        for (int k = 0; k < cpl; ++k) s += ip ? chunk_ip<RR_F32>(x[k], y[k]) : chunk_part<RR_F32>(x[k], y[k]);
        for (int o = 1; o < g; o <<= 1) s += __shfl_xor(s, o);
        if (ip) s = -s;
        const bool mine = gl == 0 && e < n;
        if (MODE == SPLIT_MIN) {
            // (a load first: an atomic for every candidate is 40 to 90 ps of it;
            // the value only falls, so an old one costs an atomic at most)
            if (mine && s <= __builtin_huge_val() && dbl_order(s) < a.sc.nn_bits[q])
                atomicMin(&a.sc.nn_bits[q], dbl_order(s));
        } else {
            const bool hit = mine && s <= a.sc.qth[q].r;
            const unsigned long long hm = __ballot(hit);
            wave_sync();
            if (hit) {
                const int o = kept + mbcnt(hm);
                st_q[o] = q;
                st_id[o] = id;
                st_d[o] = s;
            }
            kept += __popcll(hm);
        }
        wave_sync();
    }
    if (MODE == SPLIT_RANGE && kept > 0) split_emit(a, st_q, st_id, st_d, kept, lane);
}

// KS: 16-value steps held at a time (even); MULTI: rows of more than 16 KS
// values take several passes over a tile, the sums kept in between
template <int KS, bool MULTI, int MODE>
__global__ __launch_bounds__(256, 2) void k_scan_split(SplitArgs a) {
    constexpr int CPR = 2 * KS;       // 16-byte chunks per row and part
    constexpr int UNITS = KS / 2;     // chunks a thread splits per step
    constexpr int PART = SPLIT_TILE * CPR;
    extern __shared__ __align__(16) uint8_t smem[];
    uint4 *xt = reinterpret_cast<uint4 *>(smem); // [2 buffers][2 parts][PART]
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    double *st_d = reinterpret_cast<double *>(smem + 4 * PART * 16) + wid * SPLIT_STAGE;
    uint32_t *st_q = reinterpret_cast<uint32_t *>(smem + 4 * PART * 16 + 4 * SPLIT_STAGE * 8) + wid * 2 * SPLIT_STAGE;
    uint32_t *st_id = st_q + SPLIT_STAGE;
    const ScanPlace at = scan_place(a.sc);
    const int64_t q0 = (int64_t)at.qblock * SPLIT_Q + wid * 32;
    const int64_t p_begin = at.chunk * a.sc.chunk, p_end = min(a.sc.ix.n, p_begin + a.sc.chunk);
    if (p_begin >= p_end) return;
    const bool active = q0 < a.sc.nq; // waves without queries only help to load
    const bool ip = a.sc.ix.metric == RR_IP;
    const int cols = a.sc.ix.row_bytes / 4;
    const int nkc = MULTI ? a.kpad / (KS * 16) : 1;
    const int half = lane >> 5, l32 = lane & 31;
    auto swz = [](int row) { return KS == 8 ? row & 15 : KS == 4 ? (row >> 1) & 7 : (row >> 2) & 3; };

    f32x8 nx[UNITS];
    auto load_x = [&](int64_t p0, int kc) {
#pragma unroll
        for (int j = 0; j < UNITS; ++j) {
            const int u = tid + 256 * j, row = u / CPR, c = u % CPR;
            const int64_t p = min(p0 + row, p_end - 1);
            const int col = kc * KS * 16 + c * 8;
            if (col < cols) {
                nx[j] = *reinterpret_cast<const f32x8 *>(a.sc.ix.base + p * a.sc.ix.row_bytes + col * 4);
            } else {
                nx[j] = f32x8{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            }
        }
    };
    auto store_x = [&](int buf) {
#pragma unroll
        for (int j = 0; j < UNITS; ++j) {
            const int u = tid + 256 * j, row = u / CPR, c = u % CPR;
            uint4 h, l;
            split8(nx[j], h, l);
            const int o = row * CPR + (c ^ swz(row));
            xt[2 * buf * PART + o] = h;
            xt[(2 * buf + 1) * PART + o] = l;
        }
    };
    // A operand: lane l holds query l % 32, values 16 k + 8 (l / 32) + [0, 8)
    bf16x8 Ah[KS], Al[KS];
    auto load_q = [&](int kc) {
        const int64_t q = min(q0 + l32, a.sc.nq - 1);
        const uint16_t *r = a.qs + (size_t)q * 2 * a.kpad + kc * KS * 16 + half * 8;
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            Ah[k] = *reinterpret_cast<const bf16x8 *>(r + 16 * k);
            Al[k] = *reinterpret_cast<const bf16x8 *>(r + a.kpad + 16 * k);
        }
    };
    if (active && !MULTI) load_q(0);
    // output tile: lane l, register v holds query 8 (v / 4) + 4 (l / 32) + v % 4
    // and point l % 32
    f32x16 c0, lim;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int64_t q = q0 + 8 * (v / 4) + 4 * half + v % 4;
        c0[v] = MODE == SPLIT_MAX ? 0.f : q < a.sc.nq ? a.cinit[q] : -__builtin_huge_valf();
        lim[v] = -__builtin_huge_valf();
    }
    int scnt = 0; // staged candidates of this wave (wave-uniform)
    // the open run of dense tiles (none: run = -1)
    int64_t run = -1, run_p = 0;
    int run_n = 0;
    auto close_run = [&](int64_t end) {
        if (run >= 0 && lane == 0)
            a.dense[run] = make_uint4((uint32_t)(q0 / 32), (uint32_t)run_p, (uint32_t)end, 0u);
        run = -1;
    };
    f32x16 acc[2];
    load_x(p_begin, 0);
    int buf = 0;
    for (int64_t p0 = p_begin; p0 < p_end; p0 += SPLIT_TILE) {
        float hx[2];
        bool pv[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int64_t p = p0 + 32 * t + l32;
            pv[t] = p < p_end;
            hx[t] = ip ? 0.f : a.sc.ix.half_norm[min(p, p_end - 1)];
            acc[t] = c0;
        }
        for (int kc = 0; kc < nkc; ++kc) {
            if (MULTI && active) load_q(kc);
            store_x(buf);
            __syncthreads();
            if (kc + 1 < nkc) load_x(p0, kc + 1);
            else if (p0 + SPLIT_TILE < p_end) load_x(p0 + SPLIT_TILE, 0);
            if (active) {
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    bf16x8 bh[2], bl[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int row = 32 * t + l32;
                        const int o = row * CPR + ((2 * k + half) ^ swz(row));
                        bh[t] = __builtin_bit_cast(bf16x8, xt[2 * buf * PART + o]);
                        bl[t] = __builtin_bit_cast(bf16x8, xt[(2 * buf + 1) * PART + o]);
                    }
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Ah[k], bh[t], acc[t], 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Ah[k], bl[t], acc[t], 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Al[k], bh[t], acc[t], 0, 0, 0);
                }
            }
            // the other buffer is free: every wave has passed this step's
            // barrier, so it is done with the step before
            buf ^= 1;
        }
        if (!active) continue;
        if (MODE == SPLIT_MAX) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
                if (pv[t]) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) lim[v] = fmaxf(lim[v], acc[t][v] - hx[t]);
                }
            continue;
        }
        unsigned long long some[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            float top = acc[t][0];
#pragma unroll
            for (int v = 1; v < 16; ++v) top = fmaxf(top, acc[t][v]);
            some[t] = __ballot(pv[t] && top >= hx[t]);
        }
        // (so many candidates lie on half of the lanes' columns or more, but for
        // the most uneven tiles)
        bool dense = false;
        if (a.dense_cap > 0 && __popcll(some[0]) + __popcll(some[1]) >= 64) {
            int n = 0;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) n += __popcll(__ballot(pv[t] && acc[t][v] >= hx[t]));
            dense = n >= (run >= 0 ? SPLIT_STAY : SPLIT_DENSE);
        }
        if (dense) {
            if (run >= 0 && run_n == a.run_max) close_run(p0);
            if (run < 0) {
                unsigned long long r = 0;
                if (lane == 0) r = atomicAdd(a.dense_cnt, 1ull);
                r = (unsigned long long)uniform64((int64_t)r);
                dense = (int64_t)r < a.dense_cap; // else the tile is decided like any other
                if (dense) {
                    run = (int64_t)r;
                    run_p = p0;
                    run_n = 0;
                }
            }
            if (dense) {
                ++run_n;
                continue;
            }
        }
        if (run >= 0) close_run(p0);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (!some[t]) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const bool cand = pv[t] && acc[t][v] >= hx[t];
                const unsigned long long cm = __ballot(cand);
                if (!cm) continue;
                const int nc = __popcll(cm);
                if (scnt + nc > SPLIT_STAGE) {
                    split_flush<MODE>(a, st_q, st_id, st_d, scnt, lane);
                    scnt = 0;
                }
                if (cand) {
                    const int o = scnt + mbcnt(cm);
                    st_q[o] = (uint32_t)(q0 + 8 * (v / 4) + 4 * half + v % 4);
                    st_id[o] = (uint32_t)(p0 + 32 * t + l32);
                }
                scnt += nc;
            }
        }
    }
    if (!active) return;
    if (MODE == SPLIT_MAX) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            float m = lim[v];
            for (int o = 1; o < 32; o <<= 1) m = fmaxf(m, __shfl_xor(m, o));
            const int64_t q = q0 + 8 * (v / 4) + 4 * half + v % 4;
            if (l32 == 0 && q < a.sc.nq) atomicMax(&a.best[q], flt_order(m));
        }
    } else {
        close_run(p_end);
        if (scnt > 0) split_flush<MODE>(a, st_q, st_id, st_d, scnt, lane);
    }
}

// A group of chunks is summed (its pairs' sums in `v`): neighbouring groups
// first, then neighbouring pairs of groups, ...  S[i] holds the last sums of 2^i
// groups that wait for their neighbours'; group l completes the levels of its
// trailing ones.  After the last group v holds the whole sums.
template <int I, int L> __device__ __forceinline__ void dense_merge(double (&S)[L][8], double (&v)[8], int l, int low) {
    if constexpr (I < L) {
        if (((I < 3 ? low : l) >> I) & 1) { // low: l's last three bits
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] += S[I][i];
            dense_merge<I + 1, L>(S, v, l, low);
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) S[I][i] = v[i];
        }
    }
}

// The runs of dense tiles, every pair in FP64 from the float32 rows: 2^L groups
// of cpl chunks a row, a group's chunks in their order and then halves
// together, which are the sums of eval64 to the last bit.  A workgroup takes a
// tile of 32 queries and 64 points through LDS, 128 bytes of each row at a time
// (loaded a step ahead); a lane has 2 queries and 4 points, so that 6 chunks
// read serve 8 pairs.  Bound by the FP64 vector units: 8 pairs of a chunk are
// 24 conversions, 32 subtractions and 32 products, 7.3 and 58 ps a pair of 96
// and 768 values without a wait; it takes 13 and 95 (the FP64 scan: 16 and 145).
// With 6 chunks read from the L1 cache instead, 27 and 195.  Calls in which
// every pair passes the filter, FP64 scan / candidates one by one / now:
// nearest distances of 2,000 queries x 200,000 x 96 6.6 / 34.5 / 6.0 ms, of
// 2,000 x 50,000 x 768 14.4 / 70.4 / 11.1 ms, of 2,000 x 200,000 x 16 (two passes
// of the filter are half of it) 1.15 / 31 / 1.57 ms; a radius around half of
// 500 x 50,000 x 768 pairs 14.3 / 25.7 / 9.3 ms.
template <int L, bool ONE, bool IP, int MODE>
__global__ __launch_bounds__(256, L <= 2 && MODE == SPLIT_MIN ? 3 : 2) void k_split_dense(SplitArgs a) {
    // (ONE: a group is one chunk, and the order of the sums is known while the
    // loop over a step's chunks is unrolled)
    constexpr int ROWS = SPLIT_TILE + 32; // points, then queries
    constexpr int STAGE = MODE == SPLIT_RANGE ? 320 : 1;
    __shared__ uint4 xt[2][ROWS * 8];
    __shared__ double sd[4][STAGE];
    __shared__ uint32_t sq[4][STAGE], si[4][STAGE];
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int64_t runs = min((int64_t)*a.dense_cnt, a.dense_cap);
    const size_t rb = a.sc.ix.row_bytes;
    const int chunks = a.sc.ix.row_bytes / 16, cpl = a.cpl;
    // (16 lanes that read one chunk column of 16 rows fall on different banks)
    auto place = [](int row, int c) { return row * 8 + (c ^ ((row >> 1) & 7)); };
    int buf = 0;
    for (int64_t it = blockIdx.x; it < runs; it += gridDim.x) {
        const uint4 r = a.dense[it];
        const int64_t q0 = (int64_t)r.x * 32, end = r.z;
        const int ql = wid * 8 + (lane >> 4) * 2, pl = lane & 15; // of the lane, in the tile
        double lim[2]; // the radius, or the smallest distance so far
#pragma unroll
        for (int i = 0; i < 2; ++i)
            lim[i] = MODE == SPLIT_RANGE ? a.sc.qth[min(q0 + ql + i, a.sc.nq - 1)].r : __builtin_huge_val();
        uint4 nx[3];
        auto load = [&](int64_t p0, int c0) {
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int row = (tid + 256 * j) / 8, c = c0 + tid % 8;
                const uint8_t *x = j < 2 ? a.sc.ix.base + min(p0 + row, a.sc.ix.n - 1) * rb
                                         : a.sc.qpad + min(q0 + row - SPLIT_TILE, a.sc.nq - 1) * rb;
                nx[j] = c < chunks ? *reinterpret_cast<const uint4 *>(x + c * 16) : make_uint4(0u, 0u, 0u, 0u);
            }
        };
        load(r.y, 0);
        int n = 0; // staged hits (wave-uniform)
        for (int64_t p0 = r.y; p0 < end; p0 += SPLIT_TILE) {
            double S[L][8], v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = 0.0;
            int k = 0, l = 0; // chunks of the open group, its number
            for (int c0 = 0; c0 < chunks; c0 += 8, buf ^= 1) {
                // (the other buffer is free: every wave that has passed this
                // step's barrier is done with the step before)
#pragma unroll
                for (int j = 0; j < 3; ++j) xt[buf][place((tid + 256 * j) / 8, tid % 8)] = nx[j];
                __syncthreads();
                if (c0 + 8 < chunks) load(p0, c0 + 8);
                else if (p0 + SPLIT_TILE < end) load(p0 + SPLIT_TILE, 0);
                auto add = [&](int c) __attribute__((always_inline)) {
                    uint4 y[2], x[4];
#pragma unroll
                    for (int i = 0; i < 2; ++i) y[i] = xt[buf][place(SPLIT_TILE + ql + i, c)];
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = xt[buf][place(16 * j + pl, c)];
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            v[4 * i + j] += IP ? chunk_ip<RR_F32>(x[j], y[i]) : chunk_part<RR_F32>(x[j], y[i]);
                };
                auto close = [&](int low) __attribute__((always_inline)) {
                    dense_merge<0, L>(S, v, l, low);
                    if (++l < (1 << L)) {
#pragma unroll
                        for (int i = 0; i < 8; ++i) v[i] = 0.0;
                    }
                };
                if constexpr (ONE) {
#pragma unroll
                    for (int c = 0; c < (L == 2 ? 4 : 8); ++c) {
                        add(c);
                        close(c);
                    }
                } else {
                    const int m = min(8, chunks - c0);
#pragma unroll 2
                    for (int c = 0; c < m; ++c) {
                        add(c);
                        if (++k == cpl) {
                            close(l & 7);
                            k = 0;
                        }
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int64_t q = q0 + ql + i;
                bool hit[4];
                unsigned long long hm[4];
                int nh = 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double d = IP ? -v[4 * i + j] : v[4 * i + j];
                    hit[j] = q < a.sc.nq && p0 + 16 * j + pl < end && (MODE == SPLIT_MIN ? d < lim[i] : d <= lim[i]);
                    if (MODE == SPLIT_MIN) {
                        lim[i] = hit[j] ? d : lim[i];
                    } else {
                        hm[j] = __ballot(hit[j]);
                        nh += __popcll(hm[j]);
                    }
                }
                if (MODE == SPLIT_MIN || nh == 0) continue;
                if (n + nh > STAGE) {
                    split_emit(a, sq[wid], si[wid], sd[wid], n, lane);
                    n = 0;
                }
                // the hits of a query (16 lanes, four points each) one after the other
                const int sh = lane & 48;
                int o = n;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    o += __popcll(hm[j] & ((1ull << sh) - 1ull)) + __popc((unsigned)(hm[j] >> sh) & ((1u << pl) - 1u));
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (hit[j]) {
                        sq[wid][o] = (uint32_t)q;
                        si[wid][o] = (uint32_t)(p0 + 16 * j + pl);
                        sd[wid][o] = IP ? -v[4 * i + j] : v[4 * i + j];
                        ++o;
                    }
                n += nh;
            }
        }
        if (MODE == SPLIT_MIN) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                double m = lim[i];
                for (int o = 1; o < 16; o <<= 1) m = fmin(m, __shfl_xor(m, o));
                if (pl == 0 && q0 + ql + i < a.sc.nq) atomicMin(&a.sc.nn_bits[q0 + ql + i], dbl_order(m));
            }
        } else if (n > 0) {
            split_emit(a, sq[wid], si[wid], sd[wid], n, lane);
        }
    }
}

template <bool IP, int MODE> static hipError_t run_dense(const SplitArgs &a, hipStream_t s) {
    const dim3 grid(2 * device_cus()), block(256);
#define RR_DENSE(L)                                                                           \
    if (a.g == (1 << L)) {                                                                    \
        if (a.cpl == 1) hipLaunchKernelGGL((k_split_dense<L, true, IP, MODE>), grid, block, 0, s, a); \
        else hipLaunchKernelGGL((k_split_dense<L, false, IP, MODE>), grid, block, 0, s, a);    \
        return hipGetLastError();                                                             \
    }
    RR_DENSE(2) RR_DENSE(3) RR_DENSE(4) RR_DENSE(5) RR_DENSE(6)
#undef RR_DENSE
    return hipErrorInvalidValue;
}
template <int MODE> static hipError_t dispatch_dense(const SplitArgs &a, hipStream_t s) {
    if (a.dense_cap == 0) return hipSuccess;
    return a.sc.ix.metric == RR_IP ? run_dense<true, MODE>(a, s) : run_dense<false, MODE>(a, s);
}

// float32 squares of the base and of the products must be normal numbers:
// otherwise the FP64 scan runs
bool scan_split_ok(const DevIndex &ix) {
    return ix.dtype == RR_F32 && ix.half_norm && ix.max_norm >= 1e-12f && ix.max_norm <= 1e17f;
}

static int split_ks(int32_t d) { return d <= 32 ? 2 : d <= 64 ? 4 : d <= 96 ? 6 : 8; }
static int32_t split_kpad(int32_t d) {
    const int32_t k = split_ks(d) * 16;
    return (d + k - 1) / k * k;
}

// Runs of dense tiles that are kept: enough for every tile of up to 65,536, and
// beyond that for runs of 8 tiles with gaps between them; at 1M runs (16 MB)
// the runs get longer.  Scans of fewer pairs than SPLIT_FEW keep none: at most
// 43 us of single decisions, and one launch less.
constexpr int64_t SPLIT_FEW = 65536;
// More queries take the FP64 scan: a launch holds less than 2^32 threads, and 8
// chunks of the base for each 128 of these are 2^31
constexpr int64_t SPLIT_MOST = 1ll << 27;
struct DenseRoom {
    int64_t cap;
    int32_t run_max;
};
static DenseRoom dense_room(int64_t n, int64_t nq) {
    if (n * nq < SPLIT_FEW) return {0, 1};
    const int64_t tiles = (n + SPLIT_TILE - 1) / SPLIT_TILE * ((nq + 31) / 32);
    const int64_t cap = std::min<int64_t>({tiles, std::max<int64_t>(65536, tiles / 4), 1 << 20});
    return {cap, (int32_t)std::max<int64_t>(8, 4 * tiles / cap)};
}

// the runs and their count, then split queries, the threshold term, the slack
// and the best sum of every query
int64_t scan_ws_bytes(const DevIndex &ix, int64_t nq) {
    return scan_split_ok(ix) && nq <= SPLIT_MOST ? 16 + 16 * dense_room(ix.n, nq).cap + nq * ((int64_t)split_kpad(ix.d) * 4 + 12) : 0;
}

struct SplitWs {
    unsigned long long *dense_cnt;
    uint4 *dense;
    uint16_t *qs;
    float *cinit, *slack;
    unsigned *best;
};
static SplitWs split_ws(const DevIndex &ix, int64_t nq, uint8_t *ws) {
    SplitWs w;
    w.dense_cnt = reinterpret_cast<unsigned long long *>(ws);
    w.dense = reinterpret_cast<uint4 *>(ws + 16);
    ws += 16 + 16 * dense_room(ix.n, nq).cap;
    w.qs = reinterpret_cast<uint16_t *>(ws);
    w.cinit = reinterpret_cast<float *>(ws + nq * (int64_t)split_kpad(ix.d) * 4);
    w.slack = w.cinit + nq;
    w.best = reinterpret_cast<unsigned *>(w.slack + nq);
    return w;
}

template <int KS, bool MULTI, int MODE> static hipError_t run_split(SplitArgs &a, hipStream_t s) {
    const size_t shmem = (size_t)4 * SPLIT_TILE * 2 * KS * 16 + 4 * SPLIT_STAGE * 16;
    int per_cu = 0;
    auto kern = k_scan_split<KS, MULTI, MODE>;
    const hipError_t e = kernel_occupancy((const void *)kern, 256, shmem, &per_cu);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kern, dim3((unsigned)a.groups), dim3(256), shmem, s, a);
    return hipGetLastError();
}

template <int MODE> static hipError_t dispatch_split(SplitArgs &a, hipStream_t s) {
    switch (split_ks(a.sc.ix.d)) {
    case 2: return run_split<2, false, MODE>(a, s);
    case 4: return run_split<4, false, MODE>(a, s);
    case 6: return run_split<6, false, MODE>(a, s);
    default: return a.kpad <= 128 ? run_split<8, false, MODE>(a, s) : run_split<8, true, MODE>(a, s);
    }
}

static SplitWs split_args(const ScanArgs &sc, uint8_t *ws, SplitArgs &a) {
    const SplitWs w = split_ws(sc.ix, sc.nq, ws);
    a.sc = sc;
    a.dense = w.dense;
    // (a range scan's count lies behind its hit count: the caller copies both)
    a.dense_cnt = sc.item_cursor ? sc.item_cursor + 1 : w.dense_cnt;
    const DenseRoom room = dense_room(sc.ix.n, sc.nq);
    a.dense_cap = room.cap;
    a.run_max = room.run_max;
    a.qs = w.qs;
    a.cinit = w.cinit;
    a.best = w.best;
    a.kpad = split_kpad(sc.ix.d);
    row_split(sc.ix.row_bytes, &a.cpl, &a.g);
    a.sc.qblocks = (int32_t)((sc.nq + SPLIT_Q - 1) / SPLIT_Q);
    const ScanSplit sp = scan_split((sc.ix.n + SPLIT_TILE - 1) / SPLIT_TILE, a.sc.qblocks);
    a.sc.chunk = sp.chunk * SPLIT_TILE;
    a.sc.xcd_bits = sp.xcd_bits;
    a.groups = sp.groups(a.sc.qblocks);
    return w;
}

static hipError_t split_setup(const ScanArgs &sc, uint8_t *ws, SplitArgs &a, SplitWs &w, hipStream_t s) {
    w = split_args(sc, ws, a);
    hipLaunchKernelGGL(k_split_prep, dim3((unsigned)std::min<int64_t>((sc.nq + 3) / 4, 1 << 20)), dim3(256), 0, s, sc.qpad, sc.qth, sc.nq,
                       sc.ix.row_bytes, sc.ix.d, a.kpad, (double)sc.ix.max_norm, (int)(sc.ix.metric == RR_IP),
                       w.qs, w.cinit, w.slack, w.best, a.dense_cnt);
    return hipGetLastError();
}

hipError_t launch_split_range(const ScanArgs &sc, uint8_t *ws, hipStream_t s) {
    SplitArgs a;
    SplitWs w;
    const hipError_t e = split_setup(sc, ws, a, w, s);
    return e != hipSuccess ? e : dispatch_split<SPLIT_RANGE>(a, s);
}

hipError_t launch_split_range_dense(const ScanArgs &sc, uint8_t *ws, hipStream_t s) {
    SplitArgs a;
    split_args(sc, ws, a);
    return dispatch_dense<SPLIT_RANGE>(a, s);
}

// Two passes: the largest approximate sum of every query, then the pairs
// within two slacks of it, decided in FP64.  One pass with a running bound
// would hand over every record of every lane's sequence (about 80 per query
// and chunk) instead of a few pairs per query.
hipError_t launch_split_nn(const ScanArgs &sc, uint8_t *ws, hipStream_t s) {
    SplitArgs a;
    SplitWs w;
    ScanArgs sc0 = sc;
    sc0.qth = nullptr;
    hipError_t e = split_setup(sc0, ws, a, w, s);
    if (e != hipSuccess) return e;
    e = dispatch_split<SPLIT_MAX>(a, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_split_best, dim3((unsigned)((sc.nq + 255) / 256)), dim3(256), 0, s, w.best, w.slack,
                       sc.nq, w.cinit, sc.nn_bits);
    e = hipGetLastError();
    if (e == hipSuccess) e = dispatch_split<SPLIT_MIN>(a, s);
    return e != hipSuccess ? e : dispatch_dense<SPLIT_MIN>(a, s);
}

} // namespace rr
