// rr_scan.hip -- dense query x base scan on the matrix cores (ground truth).
//
// Definition 2.1 evaluated for every pair: K_q = { p : d(p, q) <= r_q }, plus
// the per-query nearest-neighbour distance used to choose radii.  The scan is
// a dense contraction Q X^T, so it runs on MFMA:
//  * uint8 / int8: v_mfma_i32_16x16x64_i8 (nearest distances) and
//    v_mfma_i32_32x32x32_i8 (range).  uint8 values are shifted by -128
//    (x ^ 0x80) into int8; squared distances are shift invariant, so
//    d = |q'|^2 + |x'|^2 - 2 q'.x' is exact in int32.
//  * float32: a bfloat16 filter with an exact FP64 decision
//    (rr_scan_f32.hip); data whose squares leave the float32 range takes
//    k_scan_f32 here, v_mfma_f64_16x16x4f64 on the values widened to FP64,
//    d = |q|^2 + |x|^2 - 2 q.x in FP64.
// The negated inner product (Section 2) uses the same products: float32
// d = -q.x; integer data keeps the search's unsigned key key_off - q.x,
// where for uint8 q.x = q'.x' + 128 (sum q + sum x) - 128^2 P over the P
// padded coordinates (padding is 0 before the shift).
// k_scan_int: each wave keeps QT (8 or 4) tiles of 16 queries in registers (A operand) and
// streams 16-point base tiles (B operand); the four waves of a workgroup
// share the base tiles through the L1 cache.  Output tile layout of the int8
// 16x16x64 MFMA: lane l, register v holds row 4*(l/16)+v, column l%16.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>

#include "rr_scan.h"

namespace rr {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

// 16-query tiles per wave: 8 for rows up to 128 bytes (twice the MFMA work
// per base tile loaded), 4 for longer rows, whose A operands would not fit
constexpr int scan_qt(int ks) { return ks <= 2 ? 8 : 4; }
constexpr int SCAP = 256; // range hits staged in LDS per wave before a flush

// Range hits of one wave, staged in its own LDS slice and appended to the
// item arrays in one block: one cursor atomic per flush instead of one per
// ballot (a single device-wide counter serialises under many writers).
// Every lane of the wave calls it with the same n.
template <typename DT>
__device__ __forceinline__ void flush_hits(const ScanArgs &a, const uint32_t *st_task, const uint32_t *st_id,
                                           const DT *st_dist, int n, int lane) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(a.item_cursor, (unsigned long long)n);
    base = __shfl(base, 0);
    for (int i = lane; i < n; i += 64) {
        const int64_t pos = (int64_t)base + i;
        const uint32_t q = st_task[i];
        if (pos < a.item_cap) {
            a.item_key[pos] = ((unsigned long long)q << 32) | st_id[i];
            ((DT *)a.item_dist)[pos] = st_dist[i];
            atomicAdd(&a.task_cnt[q], 1ull);
        } else {
            atomicOr(a.overflow, 64ull);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t shift_u8(uint32_t w) { return w ^ 0x80808080u; }

// the value of lane (lane ^ 16) by ds_swizzle in bit mode, and of lane
// (lane ^ 32) by the permlane32 swap (lanes 32-63 of one copy trade places
// with lanes 0-31 of another), without ds_bpermute's address arithmetic and
// LDS round trip; every lane of the wave must be active
__device__ __forceinline__ int xor16(int v) { return __builtin_amdgcn_ds_swizzle(v, 0x401F); }
__device__ __forceinline__ int xor32(int v) {
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return (int)((threadIdx.x & 32) ? r[0] : r[1]);
}

// running sum of the 16 unsigned bytes of v
__device__ __forceinline__ int row_sum_u8(uint4 v, int s) {
    unsigned t = __builtin_amdgcn_udot4(v.x, 0x01010101u, (unsigned)s, false);
    t = __builtin_amdgcn_udot4(v.y, 0x01010101u, t, false);
    t = __builtin_amdgcn_udot4(v.z, 0x01010101u, t, false);
    t = __builtin_amdgcn_udot4(v.w, 0x01010101u, t, false);
    return (int)t;
}

// nearest distance of every query, integer rows
template <int DTYPE, int KS, bool IP, int QT>
__global__ __launch_bounds__(256) void k_scan_int(ScanArgs a) {
    const int lane = threadIdx.x & 63;
    const int wid = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    constexpr int ks_n = KS; // 64-byte K steps per row
    const int64_t q0 = ((int64_t)blockIdx.x * 4 + wid) * (QT * 16);
    const int64_t p_begin = (int64_t)blockIdx.y * a.chunk;
    const int64_t p_end = min(a.ix.n, p_begin + a.chunk);
    if (q0 >= a.nq || p_begin >= p_end) return;
    constexpr int KSMAX = KS;
    v4i A[QT][KSMAX];
    int qn_own[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        const int64_t q = min(q0 + t * 16 + row, a.nq - 1);
        int s = 0;
#pragma unroll
        for (int ks = 0; ks < KSMAX; ++ks) {
            if (ks < ks_n) {
                uint4 v = *reinterpret_cast<const uint4 *>(a.qpad + q * a.ix.row_bytes + ks * 64 + grp * 16);
                if (IP && DTYPE == RR_U8) s = row_sum_u8(v, s);
                if (DTYPE == RR_U8) {
                    v.x = shift_u8(v.x);
                    v.y = shift_u8(v.y);
                    v.z = shift_u8(v.z);
                    v.w = shift_u8(v.w);
                }
                A[t][ks] = v4i{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
                if (!IP) {
                    s = __builtin_amdgcn_sdot4((int)v.x, (int)v.x, s, false);
                    s = __builtin_amdgcn_sdot4((int)v.y, (int)v.y, s, false);
                    s = __builtin_amdgcn_sdot4((int)v.z, (int)v.z, s, false);
                    s = __builtin_amdgcn_sdot4((int)v.w, (int)v.w, s, false);
                }
            }
        }
        // zero padding becomes -128 after the uint8 shift in queries and base
        // rows alike, so padded coordinates add (q'-x')^2 = 0 to the distance
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        // lanes with row == i hold |q_i'|^2, or for the inner product the
        // query part of the key: key_off (+ 128^2 P - 128 sum q for uint8)
        if (IP)
            s = (int)((uint32_t)a.ix.key_off +
                      (DTYPE == RR_U8 ? (uint32_t)(16384 * KS * 64) - 128u * (uint32_t)s : 0u));
        qn_own[t] = s;
    }
    // Every distance (or key) is qn + part with the query's constant qn and
    // part = |x'|^2 - 2 q'.x' (inner product: the base row's part - q.x),
    // exact in int32.  The loop keeps the largest neg = -part = 2 q'.x' -
    // |x'|^2 (one shift-add and one maximum per element).
    int lim[QT][4]; // the largest neg so far
#pragma unroll
    for (int t = 0; t < QT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) lim[t][v] = INT_MIN;

    // the next tile's rows are loaded while the current one is multiplied
    // (clamped to the chunk's last row, so every load is in bounds)
    uint4 nxt[KSMAX];
    {
        const uint8_t *xr = a.ix.base + min(p_begin + row, p_end - 1) * a.ix.row_bytes + grp * 16;
#pragma unroll
        for (int ks = 0; ks < KSMAX; ++ks) nxt[ks] = *reinterpret_cast<const uint4 *>(xr + ks * 64);
    }
    for (int64_t p0 = p_begin; p0 < p_end; p0 += 16) {
        uint4 cur[KSMAX];
#pragma unroll
        for (int ks = 0; ks < KSMAX; ++ks) cur[ks] = nxt[ks];
        {
            const uint8_t *xr = a.ix.base + min(p0 + 16 + row, p_end - 1) * a.ix.row_bytes + grp * 16;
#pragma unroll
            for (int ks = 0; ks < KSMAX; ++ks) nxt[ks] = *reinterpret_cast<const uint4 *>(xr + ks * 64);
        }
        v4i B[KSMAX];
        int xs = 0;
#pragma unroll
        for (int ks = 0; ks < KSMAX; ++ks) {
            if (ks < ks_n) {
                uint4 v = cur[ks];
                if (IP && DTYPE == RR_U8) xs = row_sum_u8(v, xs);
                if (DTYPE == RR_U8) {
                    v.x = shift_u8(v.x);
                    v.y = shift_u8(v.y);
                    v.z = shift_u8(v.z);
                    v.w = shift_u8(v.w);
                }
                B[ks] = v4i{(int)v.x, (int)v.y, (int)v.z, (int)v.w};
                if (!IP) {
                    xs = __builtin_amdgcn_sdot4((int)v.x, (int)v.x, xs, false);
                    xs = __builtin_amdgcn_sdot4((int)v.y, (int)v.y, xs, false);
                    xs = __builtin_amdgcn_sdot4((int)v.z, (int)v.z, xs, false);
                    xs = __builtin_amdgcn_sdot4((int)v.w, (int)v.w, xs, false);
                }
            }
        }
        xs += xor16(xs);
        xs += xor32(xs);
        if (IP) xs = -128 * xs; // the base row's part of the uint8 key (0 for int8)
        int nxs = -xs;
        // opaque to the optimiser, so that 2 acc + nxs stays one shift-add
        // instead of being refolded into a shift and a subtraction
        asm volatile("" : "+v"(nxs));
#pragma unroll
        for (int t = 0; t < QT; ++t) {
            v4i acc = {0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KSMAX; ++ks)
                if (ks < ks_n) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[t][ks], B[ks], acc, 0, 0, 0);
            // rows past the chunk repeat its last row, which leaves the
            // maximum unchanged, so no validity test is needed
#pragma unroll
            for (int v = 0; v < 4; ++v) lim[t][v] = max(lim[t][v], IP ? acc[v] + nxs : 2 * acc[v] + nxs);
        }
    }
    {
#pragma unroll
        for (int t = 0; t < QT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                int b = lim[t][v];
#pragma unroll
                for (int m = 1; m < 16; m <<= 1) b = max(b, __shfl_xor(b, m));
                const uint32_t qn = (uint32_t)__shfl(qn_own[t], 4 * grp + v);
                const int64_t q = q0 + t * 16 + 4 * grp + v;
                // every chunk has at least one valid row, so b was raised
                if (row == 0 && q < a.nq && b != INT_MIN)
                    atomicMin(&a.nn_bits[q], (unsigned long long)(qn - (uint32_t)b));
            }
    }
}

// Range scan of integer rows, v_mfma_i32_32x32x32_i8.  The four waves of a
// workgroup stream 16 KB of base rows at a time through LDS (loaded one step
// ahead; 16-byte chunks at a place xored by the row, so the lanes that read a
// chunk column fall on different banks) and each multiplies them with QT tiles
// of 32 queries that it holds in registers.
// With lim = |q'|^2 - r a pair is a hit iff 2 q'.x' - |x'|^2 >= lim, and only
// if q'.x' - floor(|x'|^2 / 2) >= floor(lim / 2): a lane's column is one
// query, the sums start at the rows' half of the test (16 registers, shared by
// the query tiles; the loading threads put it in LDS beside the rows), and
// 16 outputs take one maximum and one compare.  A tile with a hit is
// multiplied again and decided by the first test, so nothing but the maximum
// has to outlive its tile.  Inner product: the same without the halving.
// Bound by the matrix cores: 10,000 queries x 1M x 128 (2.56 T operations) are
// 0.5 ms at the 5 POP/s dense peak, about 1.0 ms at the share of its peak that
// a large bf16 product reaches.  16x16 tiles, with a shift-add, a compare
// and an or for every output, took 1.74 ms; query bounds in the sums' start
// (64 registers) and rows loaded by each wave for itself 1.50 ms, with
// two query tiles a wave 2.47 ms; this one 1.32 ms, of which the 160,000
// hits are 0.15 ms (with 677,000 hits 1.78 -> 1.61 ms).
// Output tile: lane l, register v holds row 8 (v / 4) + 4 (l / 32) + v % 4,
// query l % 32.
typedef int v16i __attribute__((ext_vector_type(16)));
constexpr int range_qt(int ks) { return ks <= 6 ? 4 : ks <= 12 ? 2 : 1; }
constexpr int range_tile(int ks) { return ks <= 4 ? 128 : ks <= 8 ? 64 : 32; } // base points per step
constexpr int range_waves(int ks) { return ks <= 2 ? 3 : 2; }                  // per SIMD, as registers allow

template <int DTYPE, int KS, bool IP, int QT>
__global__ __launch_bounds__(256, range_waves(KS)) void k_scan_range(ScanArgs a) {
    constexpr int CPR = 2 * KS;                   // 16-byte chunks per row
    constexpr int TPR = CPR % 8 == 0 ? 8 : 4;     // threads that load a row together
    constexpr int TILE = range_tile(KS), PASS = 256 / TPR;
    constexpr int ROWS = TILE / PASS, COLS = CPR / TPR; // rows and chunks of a thread per step
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int l32 = lane & 31, half = lane >> 5;
    const ScanPlace at = scan_place(a);
    // up to QT * 32 queries: every wave takes them all and a fourth of the points
    const bool few = a.nq <= QT * 32;
    const int64_t q0 = few ? 0 : ((int64_t)at.qblock * 4 + wid) * (QT * 32);
    const int sub0 = few ? wid * 32 : 0, sub_step = few ? 128 : 32;
    const int64_t p_begin = at.chunk * a.chunk;
    const int64_t p_end = min(a.ix.n, p_begin + a.chunk);
    if (p_begin >= p_end) return;
    const bool active = q0 < a.nq; // waves without queries only help to load
    __shared__ uint4 xt[2][TILE * CPR];
    __shared__ int xstart[2][TILE], xsum[2][TILE];
    auto place = [](int row, int c) {
        return row * CPR + (c ^ (CPR % 16 == 0 ? row & 15 : CPR % 8 == 0 ? (row >> 1) & 7 : (row >> 2) & 3));
    };
    __shared__ uint32_t stage[4 * 3 * SCAP];
    uint32_t *st_task = stage + wid * 3 * SCAP, *st_id = st_task + SCAP, *st_dist = st_id + SCAP;
    int scnt = 0; // staged hits of this wave (wave-uniform)
    // row sums: squares of the shifted values, or for the uint8 inner product
    // the plain values
    auto part = [](uint4 v, uint4 w, int s) {
        if (IP) return DTYPE == RR_U8 ? row_sum_u8(v, s) : 0;
        s = __builtin_amdgcn_sdot4((int)w.x, (int)w.x, s, false);
        s = __builtin_amdgcn_sdot4((int)w.y, (int)w.y, s, false);
        s = __builtin_amdgcn_sdot4((int)w.z, (int)w.z, s, false);
        return __builtin_amdgcn_sdot4((int)w.w, (int)w.w, s, false);
    };
    auto shifted = [](uint4 v) {
        return DTYPE == RR_U8 ? make_uint4(shift_u8(v.x), shift_u8(v.y), shift_u8(v.z), shift_u8(v.w)) : v;
    };
    v4i Q[QT][KS];
    int qn[QT], lim[QT]; // of the lane's query: its part of the distance, its bound
#pragma unroll
    for (int t = 0; t < QT; ++t) {
        const int64_t q = q0 + t * 32 + l32, qc = min(q, a.nq - 1);
        int s = 0;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const uint4 v = *reinterpret_cast<const uint4 *>(a.qpad + qc * a.ix.row_bytes + ks * 32 + half * 16);
            const uint4 w = shifted(v);
            s = part(v, w, s);
            Q[t][ks] = v4i{(int)w.x, (int)w.y, (int)w.z, (int)w.w};
        }
        s += xor32(s);
        if (IP)
            s = (int)((uint32_t)a.ix.key_off +
                      (DTYPE == RR_U8 ? (uint32_t)(16384 * KS * 32) - 128u * (uint32_t)s : 0u));
        qn[t] = s;
        // every sum below is under 2^26 in magnitude (d <= 512): bounds clamped
        // at -2^28 and 2^30 decide the same; queries past nq get 2^30
        lim[t] = q < a.nq ? (int)max(-(int64_t)(1 << 28), min((int64_t)(1 << 30), (int64_t)s - a.qth[qc].r_int))
                          : 1 << 30;
    }
    uint4 nxt[ROWS][COLS];
    const int lrow = tid / TPR, lcol = tid % TPR;
    auto load = [&](int64_t p0) {
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
#pragma unroll
            for (int j = 0; j < COLS; ++j)
                nxt[i][j] = *reinterpret_cast<const uint4 *>(
                    a.ix.base + min(p0 + i * PASS + lrow, p_end - 1) * a.ix.row_bytes + (lcol + j * TPR) * 16);
    };
    load(p_begin);
    int buf = 0;
    for (int64_t s0 = p_begin; s0 < p_end; s0 += TILE, buf ^= 1) {
        // (a wave that has passed this barrier is done with the step before, so
        // the next step may write the other buffer)
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            const int row = i * PASS + lrow;
            int s = 0;
#pragma unroll
            for (int j = 0; j < COLS; ++j) {
                const uint4 w = shifted(nxt[i][j]);
                s = part(nxt[i][j], w, s);
                xt[buf][place(row, lcol + j * TPR)] = w;
            }
            s += __builtin_amdgcn_update_dpp(0, s, 0xB1, 0xf, 0xf, true); // lane ^ 1
            s += __builtin_amdgcn_update_dpp(0, s, 0x4E, 0xf, 0xf, true); // lane ^ 2
            if (TPR == 8) s += __builtin_amdgcn_update_dpp(0, s, 0x141, 0xf, 0xf, true); // the other four of eight
            if (lcol == 0) {
                // rows past the chunk (copies of its last row) never pass
                xstart[buf][row] = s0 + row < p_end ? (IP ? 128 * s : -(s >> 1)) : -(1 << 29);
                xsum[buf][row] = s;
            }
        }
        __syncthreads();
        if (s0 + TILE < p_end) load(s0 + TILE);
        if (!active) continue;
        for (int sub = sub0; sub < TILE && s0 + sub < p_end; sub += sub_step) {
            v4i X[KS];
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const uint4 w = xt[buf][place(sub + l32, 2 * ks + half)];
                X[ks] = v4i{(int)w.x, (int)w.y, (int)w.z, (int)w.w};
            }
            // the lane's 16 rows of the output tile
            auto rows16 = [&](const int *of) {
                v16i r;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int4 w = *reinterpret_cast<const int4 *>(of + sub + 8 * g + 4 * half);
                    r[4 * g] = w.x, r[4 * g + 1] = w.y, r[4 * g + 2] = w.z, r[4 * g + 3] = w.w;
                }
                return r;
            };
            const v16i start = rows16(xstart[buf]);
            auto sums = [&](int t) {
                v16i acc = start;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(X[ks], Q[t][ks], acc, 0, 0, 0);
                return acc;
            };
            unsigned long long some[QT], any = 0ull;
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                const v16i acc = sums(t);
                int top = acc[0];
#pragma unroll
                for (int v = 1; v < 16; ++v) top = max(top, acc[v]);
                some[t] = __ballot(top >= (IP ? lim[t] : lim[t] >> 1));
                any |= some[t];
            }
            if (!any) continue;
#pragma unroll
            for (int t = 0; t < QT; ++t) {
                if (!some[t]) continue;
                const v16i acc = sums(t), xs = rows16(xsum[buf]);
                int h4 = sub + 4 * half;
                asm volatile("" : "+v"(h4)); // (sixteen sums with it would be kept through the loop)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int row = h4 + 8 * (v / 4) + v % 4;
                    // q'.x' and the row's part, or 2 q'.x' - |x'|^2
                    const int val = IP ? acc[v] : 2 * acc[v] - (xs[v] & 1);
                    const bool hit = val >= lim[t];
                    const unsigned long long hm = __ballot(hit);
                    if (hm) {
                        const int nh = __popcll(hm);
                        if (scnt + nh > SCAP) {
                            flush_hits(a, st_task, st_id, st_dist, scnt, lane);
                            scnt = 0;
                        }
                        if (hit) {
                            const int slot = scnt + (int)__builtin_amdgcn_mbcnt_hi(
                                (unsigned)(hm >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)hm, 0u));
                            st_task[slot] = (uint32_t)(q0 + t * 32 + l32);
                            st_id[slot] = (uint32_t)(s0 + row);
                            st_dist[slot] = (uint32_t)qn[t] - (uint32_t)val;
                        }
                        scnt += nh;
                    }
                }
            }
        }
    }
    if (scnt > 0) flush_hits(a, st_task, st_id, st_dist, scnt, lane);
}

// float32 data: FP64 MFMA (16x16x4).  A: lane l holds q[i=l%16][k=4s+l/16];
// B: lane l holds x[j=l%16][k=4s+l/16].  The FP64 output tile differs from
// the integer one: lane l, register v holds row (l/16) + 4v, column l%16.
#define F64_ROW(grp, v) ((grp) + 4 * (v))
template <bool IP, int MODE>
__global__ __launch_bounds__(256) void k_scan_f32(ScanArgs a) {
    constexpr int mode = MODE;
    const int lane = threadIdx.x & 63;
    const int wid = threadIdx.x >> 6;
    const int row = lane & 15, grp = lane >> 4;
    const int d = a.ix.d;
    const int ksteps = (d + 3) / 4;
    constexpr int QTF = 2;
    const int64_t q0 = ((int64_t)blockIdx.x * 4 + wid) * (QTF * 16);
    const int64_t p_begin = (int64_t)blockIdx.y * a.chunk;
    const int64_t p_end = min(a.ix.n, p_begin + a.chunk);
    if (q0 >= a.nq || p_begin >= p_end) return;
    __shared__ uint32_t stage_ti[MODE == SCAN_RANGE ? 4 * 2 * SCAP : 1];
    __shared__ double stage_d[MODE == SCAN_RANGE ? 4 * SCAP : 1];
    uint32_t *st_task = stage_ti + wid * 2 * SCAP, *st_id = st_task + SCAP;
    double *st_dist = stage_d + wid * SCAP;
    int scnt = 0; // staged hits of this wave (wave-uniform)
    double qn_own[QTF];
    for (int t = 0; t < QTF; ++t) {
        const int64_t q = min(q0 + t * 16 + row, a.nq - 1);
        const float *qr = (const float *)(a.qpad + q * a.ix.row_bytes);
        double s = 0;
        if (!IP)
            for (int k = grp; k < d; k += 4) s = fma((double)qr[k], (double)qr[k], s);
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        qn_own[t] = s;
    }
    double qn[QTF][4], rr_[QTF][4];
    double best[QTF][4];
    for (int t = 0; t < QTF; ++t)
        for (int v = 0; v < 4; ++v) {
            qn[t][v] = __shfl(qn_own[t], F64_ROW(grp, v));
            const int64_t q = q0 + t * 16 + F64_ROW(grp, v);
            // rows past nq never hit (the inner product has negative distances,
            // so no finite sentinel radius would exclude them)
            rr_[t][v] = (mode == SCAN_RANGE && q < a.nq) ? a.qth[q].r : -__builtin_huge_val();
            best[t][v] = __builtin_huge_val();
        }
    for (int64_t p0 = p_begin; p0 < p_end; p0 += 16) {
        const int64_t p = min(p0 + row, p_end - 1);
        const float *xr = (const float *)(a.ix.base + p * a.ix.row_bytes);
        v4d acc[QTF];
        for (int t = 0; t < QTF; ++t) acc[t] = v4d{0, 0, 0, 0};
        double xs = 0;
        for (int s = 0; s < ksteps; ++s) {
            const int k = 4 * s + grp;
            const double xv = k < d ? (double)xr[k] : 0.0;
            if (!IP) xs = fma(xv, xv, xs);
            for (int t = 0; t < QTF; ++t) {
                const int64_t q = min(q0 + t * 16 + row, a.nq - 1);
                const float *qr = (const float *)(a.qpad + q * a.ix.row_bytes);
                const double qv = k < d ? (double)qr[k] : 0.0;
                acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(qv, xv, acc[t], 0, 0, 0);
            }
        }
        xs += __shfl_xor(xs, 16);
        xs += __shfl_xor(xs, 32);
        const bool pvalid = p0 + row < p_end;
        for (int t = 0; t < QTF; ++t)
            for (int v = 0; v < 4; ++v) {
                double dd;
                if (IP) {
                    dd = -acc[t][v];
                } else {
                    dd = qn[t][v] + xs - 2.0 * acc[t][v];
                    if (dd < 0) dd = 0;
                }
                if (mode == SCAN_NN) {
                    if (pvalid && dd < best[t][v]) best[t][v] = dd;
                } else {
                    const int64_t qrow = q0 + t * 16 + F64_ROW(grp, v);
                    const bool hit = pvalid && qrow < a.nq && dd <= rr_[t][v];
                    const unsigned long long hm = __ballot(hit);
                    if (hm) {
                        const int nh = __popcll(hm);
                        if (scnt + nh > SCAP) {
                            flush_hits(a, st_task, st_id, st_dist, scnt, lane);
                            scnt = 0;
                        }
                        if (hit) {
                            const int slot = scnt + (int)__builtin_amdgcn_mbcnt_hi(
                                (unsigned)(hm >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)hm, 0u));
                            st_task[slot] = (uint32_t)qrow;
                            st_id[slot] = (uint32_t)(p0 + row);
                            st_dist[slot] = dd;
                        }
                        scnt += nh;
                    }
                }
            }
    }
    if (mode == SCAN_RANGE && scnt > 0) flush_hits(a, st_task, st_id, st_dist, scnt, lane);
    if (mode == SCAN_NN) {
        for (int t = 0; t < QTF; ++t)
            for (int v = 0; v < 4; ++v) {
                double b = best[t][v];
                for (int m = 1; m < 16; m <<= 1) b = fmin(b, __shfl_xor(b, m));
                const int64_t q = q0 + t * 16 + F64_ROW(grp, v);
                if (row == 0 && q < a.nq) atomicMin(&a.nn_bits[q], dbl_order(b));
            }
    }
}

__global__ void k_nn_finish(const unsigned long long *bits, int64_t nq, int dtype, int64_t key_off,
                            double *out) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = dtype == RR_F32 ? dbl_unorder(bits[i])
                                 : (double)(uint32_t)bits[i] - (double)key_off;
}

__global__ void k_identity_tasks(int32_t *task_q, int64_t nq, unsigned long long *counters) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nq;
         i += (int64_t)gridDim.x * blockDim.x)
        task_q[i] = (int32_t)i;
    if (blockIdx.x == 0 && threadIdx.x == 0) counters[CTR_TASKS] = (unsigned long long)nq;
}

template <int K>
static void launch_scan_int(const ScanArgs &a, bool ip, dim3 grid, dim3 block, hipStream_t s) {
    if (a.ix.dtype == RR_U8 && ip) hipLaunchKernelGGL((k_scan_int<RR_U8, K, true, scan_qt(K)>), grid, block, 0, s, a);
    else if (a.ix.dtype == RR_U8) hipLaunchKernelGGL((k_scan_int<RR_U8, K, false, scan_qt(K)>), grid, block, 0, s, a);
    else if (ip) hipLaunchKernelGGL((k_scan_int<RR_I8, K, true, scan_qt(K)>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_scan_int<RR_I8, K, false, scan_qt(K)>), grid, block, 0, s, a);
}

template <int K>
static void launch_scan_range(const ScanArgs &a, bool ip, dim3 grid, dim3 block, hipStream_t s) {
    constexpr int QT = range_qt(K);
    if (a.ix.dtype == RR_U8 && ip) hipLaunchKernelGGL((k_scan_range<RR_U8, K, true, QT>), grid, block, 0, s, a);
    else if (a.ix.dtype == RR_U8) hipLaunchKernelGGL((k_scan_range<RR_U8, K, false, QT>), grid, block, 0, s, a);
    else if (ip) hipLaunchKernelGGL((k_scan_range<RR_I8, K, true, QT>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_scan_range<RR_I8, K, false, QT>), grid, block, 0, s, a);
}

static hipError_t launch_scan(const ScanArgs &a0, int mode, hipStream_t s) {
    ScanArgs a = a0;
    const int qper = a.ix.dtype == RR_F32 ? 4 * 2 * 16
                     : mode == SCAN_NN    ? 4 * scan_qt(a.ix.row_bytes / 64) * 16
                                          : 4 * range_qt(a.ix.row_bytes / 32) * 32;
    const bool range_int = a.ix.dtype != RR_F32 && mode == SCAN_RANGE;
    const int64_t qblocks = (a.nq + qper - 1) / qper;
    a.qblocks = (int32_t)qblocks;
    dim3 block(256);
    const bool ip = a.ix.metric == RR_IP;
    const int ks = a.ix.row_bytes / 64;
    if (range_int) {
        const int tile = range_tile(2 * ks);
        const ScanSplit sp = scan_split((a.ix.n + tile - 1) / tile, qblocks);
        a.chunk = sp.chunk * tile;
        a.xcd_bits = sp.xcd_bits;
        const dim3 grid((unsigned)sp.groups(qblocks));
#define RR_SCAN_KS(K)                                                                         \
    if (ks == K) {                                                                            \
        launch_scan_range<2 * K>(a, ip, grid, block, s);                                      \
        return hipGetLastError();                                                             \
    }
        RR_SCAN_KS(1) RR_SCAN_KS(2) RR_SCAN_KS(3) RR_SCAN_KS(4) RR_SCAN_KS(6) RR_SCAN_KS(8)
#undef RR_SCAN_KS
        return hipErrorInvalidValue; // integer rows above 512 bytes are not scanned
    }
    // enough workgroups to fill the machine several times over
    int64_t target = 4096;
    int64_t pblocks = std::max<int64_t>(1, target / std::max<int64_t>(qblocks, 1));
    a.chunk = ((a.ix.n + pblocks - 1) / pblocks + 15) / 16 * 16;
    pblocks = (a.ix.n + a.chunk - 1) / a.chunk;
    if (pblocks > 65535) {
        pblocks = 65535;
        a.chunk = ((a.ix.n + pblocks - 1) / pblocks + 15) / 16 * 16;
        pblocks = (a.ix.n + a.chunk - 1) / a.chunk;
    }
    dim3 grid((unsigned)qblocks, (unsigned)pblocks);
    if (a.ix.dtype == RR_F32) {
        if (ip && mode == SCAN_NN) hipLaunchKernelGGL((k_scan_f32<true, SCAN_NN>), grid, block, 0, s, a);
        else if (ip) hipLaunchKernelGGL((k_scan_f32<true, SCAN_RANGE>), grid, block, 0, s, a);
        else if (mode == SCAN_NN) hipLaunchKernelGGL((k_scan_f32<false, SCAN_NN>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((k_scan_f32<false, SCAN_RANGE>), grid, block, 0, s, a);
        return hipGetLastError();
    }
#define RR_SCAN_KS(K)                                                                         \
    if (ks == K) {                                                                            \
        launch_scan_int<K>(a, ip, grid, block, s);                                            \
        return hipGetLastError();                                                             \
    }
    RR_SCAN_KS(1) RR_SCAN_KS(2) RR_SCAN_KS(3) RR_SCAN_KS(4) RR_SCAN_KS(6) RR_SCAN_KS(8)
#undef RR_SCAN_KS
    return hipErrorInvalidValue; // integer rows above 512 bytes are not scanned
}

hipError_t launch_nn_dist(const DevIndex &ix, const uint8_t *qpad, int64_t nq, double *nn,
                          unsigned long long *bits, uint8_t *ws, hipStream_t s) {
    if (nq == 0) return hipSuccess;
    ScanArgs a{};
    a.ix = ix;
    a.qpad = qpad;
    a.nq = nq;
    a.nn_bits = bits;
    hipError_t e = hipSuccess;
    if (ws && scan_split_ok(ix)) {
        e = launch_split_nn(a, ws, s);
    } else {
        e = launch_fill_u64(bits, nq, ~0ull, s);
        if (e == hipSuccess) e = launch_scan(a, SCAN_NN, s);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_nn_finish, dim3((unsigned)std::min<int64_t>((nq + 255) / 256, 4096)),
                       dim3(256), 0, s, bits, nq, ix.dtype, ix.key_off, nn);
    return hipGetLastError();
}

static ScanArgs range_args(const DevIndex &ix, const uint8_t *qpad, const QThresh *qth, int64_t nq, SearchBufs &sb) {
    ScanArgs a{};
    a.ix = ix;
    a.qpad = qpad;
    a.qth = qth;
    a.nq = nq;
    a.item_key = sb.item_key;
    a.item_dist = sb.item_dist;
    a.item_cap = sb.item_cap;
    a.item_cursor = &sb.level_cnt[0];
    a.task_cnt = sb.task_cnt;
    a.overflow = &sb.counters[CTR_OVERFLOW];
    return a;
}

hipError_t launch_brute_force_dense(const DevIndex &ix, const uint8_t *qpad, const QThresh *qth, int64_t nq,
                                    SearchBufs &sb, uint8_t *ws, hipStream_t s) {
    return launch_split_range_dense(range_args(ix, qpad, qth, nq, sb), ws, s);
}

hipError_t launch_brute_force(const DevIndex &ix, const uint8_t *qpad, const QThresh *qth,
                              int64_t nq, SearchBufs &sb, uint8_t *ws, int num_cus, hipStream_t s) {
    (void)num_cus;
    if (nq == 0) return hipSuccess;
    hipLaunchKernelGGL(k_identity_tasks, dim3((unsigned)std::min<int64_t>((nq + 255) / 256, 4096)),
                       dim3(256), 0, s, sb.task_q, nq, sb.counters);
    hipError_t e = launch_fill_u64(sb.task_cnt, nq, 0ull, s);
    if (e != hipSuccess) return e;
    e = launch_fill_u64(sb.task_evals, nq, 0ull, s);
    if (e != hipSuccess) return e;
    const ScanArgs a = range_args(ix, qpad, qth, nq, sb);
    return ws && scan_split_ok(ix) ? launch_split_range(a, ws, s) : launch_scan(a, SCAN_RANGE, s);
}

} // namespace rr
