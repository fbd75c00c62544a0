// rr_search.h -- device code of the range search (templates), shared by the
// translation units that instantiate it for each data type.
//
// One wavefront (64 lanes) runs one query's beam search (Algorithm 1) with
// the d_visited early stop (Algorithm 5).  Queries come from a device-side
// atomic queue, so a grid sized to the machine drains any batch.  Queries
// whose in-range beam reaches the expansion threshold (Algorithm 6) become
// tasks of the greedy phase (Algorithm 2).  The closure inside the ball does
// not depend on visiting order, so every frontier node of every query is an
// independent work item: where the set of a task fits in LDS one workgroup
// runs a task, and a cooperative grid runs the rest, and the large balls
// handed on, level by level over all tasks at once.
//
// Exactness of the beam on a GPU rests on two facts about Algorithm 1 under
// the total order (d, id):
//  * the b-th key of B never increases once |B| = b, so a point that was
//    evaluated and trimmed is trimmed again if it is re-inserted;
//  * therefore filtering neighbours by "ever evaluated" instead of by V gives
//    the same B, and a cache of evaluated ids that may FORGET entries (never
//    invent them) is exact as long as insertion into B removes duplicates.
// The LDS seen-cache below is such a cache.
//
// Memory traffic: a neighbour row is read by a group of G lanes, each loading
// CPL 16-byte chunks, so one load instruction covers 64/G whole rows with
// fully used 64/128-byte segments.  Distances: uint8/int8 via the 4-way dot
// instructions (|p|^2 - 2 p.q + |q|^2, exact in int32); float32 with FP64
// accumulation of the differences.
#pragma once

#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "rr_internal.h"

namespace rr {

// --------------------------------------------------------------------------
// small device helpers
// --------------------------------------------------------------------------

#define RR_IDMASK 0x7fffffffu
#define RR_VIS 0x80000000u
#define RR_EMPTY32 0xffffffffu

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ int mbcnt(unsigned long long m) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

template <typename D>
__device__ __forceinline__ bool key_less(D da, uint32_t ia, D db, uint32_t ib) {
    return da < db || (da == db && ia < ib);
}

template <typename D> __device__ __forceinline__ D dmax();
template <> __device__ __forceinline__ uint32_t dmax<uint32_t>() { return 0xffffffffu; }
template <> __device__ __forceinline__ double dmax<double>() { return __builtin_huge_val(); }
template <> __device__ __forceinline__ float dmax<float>() { return __builtin_huge_valf(); }

__device__ __forceinline__ uint32_t hash32(uint32_t x) { return x * 2654435761u; }

// LDS seen-cache of cs ids (a power of two, at least 64) in buckets of
// eight; `shift` is 32 - log2(cs / 8).  Returns true if `id` was already
// present.  A full bucket loses one of its ids to the new one (the cache
// forgets it) and `overflow` is set.  One pair of 16-byte reads decides a
// bucket where a linear probe would take up to eight dependent atomics, and
// a long search keeps its recent ids, which are the ones that come back.
__device__ __forceinline__ bool seen_insert(uint32_t *tab, int shift, uint32_t id, bool &overflow) {
    const uint32_t h = id * 2654435761u;
    uint32_t *const bk = tab + 8 * (h >> shift);
    for (;;) {
        const uint4 u = reinterpret_cast<const uint4 *>(bk)[0], v = reinterpret_cast<const uint4 *>(bk)[1];
        const uint32_t w[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
        uint32_t diff = ~0u, empty = 0u;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            diff = min(diff, w[j] ^ id);
            empty |= w[j] == RR_EMPTY32 ? 1u << j : 0u;
        }
        if (diff == 0u) return true;
        // the first empty slot from a place of the id's own, so that lanes
        // that meet in a bucket seldom want the same slot
        const uint32_t at = (h >> 4) & 7u;
        if (empty == 0u) {
            bk[at] = id;
            overflow = true;
            return false;
        }
        const uint32_t e = ((uint32_t)__ffs((int)((empty | empty << 8) >> at)) - 1u + at) & 7u;
        // another lane may take the slot first (the ids of one visit differ)
        if (atomicCAS(bk + e, RR_EMPTY32, id) == RR_EMPTY32) return false;
    }
}

// Global exact set of (task, id) keys: returns true if the key was inserted
// now, false if it was present.  `full` is set if the probe budget ran out.
// Probing reads whole 8-slot buckets (64 bytes) with plain loads and uses CAS
// only on the first slot that looked empty.  Within one search a slot only
// ever changes from empty to a key, so a stale read can only show "empty";
// the CAS then fails and reveals the key, so the set stays exact.
__device__ __forceinline__ uint64_t gset_bucket(int64_t cap_mask, unsigned long long key) {
    uint64_t h = (uint64_t)hash32((uint32_t)key ^ hash32((uint32_t)(key >> 32))) * 0x9E3779B97F4A7C15ull;
    h ^= h >> 29;
    return h & (uint64_t)cap_mask & ~7ull;
}

__device__ __forceinline__ bool gset_insert(unsigned long long *tab, int64_t cap_mask,
                                            unsigned long long key, bool &full) {
    const uint64_t b0 = gset_bucket(cap_mask, key);
#pragma unroll 1
    for (int pb = 0; pb < 16; ++pb) {
        const uint64_t b = (b0 + 8ull * (uint64_t)pb) & (uint64_t)cap_mask;
        const uint4 *bp = reinterpret_cast<const uint4 *>(tab + b);
        unsigned long long v[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint4 w = bp[j];
            v[2 * j] = ((unsigned long long)w.y << 32) | w.x;
            v[2 * j + 1] = ((unsigned long long)w.w << 32) | w.z;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (v[j] == key) return false;
            if (v[j] == ~0ull) {
                const unsigned long long old = atomicCAS(&tab[b + j], ~0ull, key);
                if (old == ~0ull) return true;
                if (old == key) return false;
            }
        }
    }
    full = true;
    return false;
}

// Two keys at once (either may be absent): both bucket reads, then both
// CASes, are in flight together.  The first four slots of each bucket decide
// the common case; anything else takes gset_insert's full probe.
// -2: key present; 0..3: first empty slot; -1: undecided
__device__ __forceinline__ int gset_scan4(uint4 w0, uint4 w1, unsigned long long key) {
    const unsigned long long v[4] = {((unsigned long long)w0.y << 32) | w0.x,
                                     ((unsigned long long)w0.w << 32) | w0.z,
                                     ((unsigned long long)w1.y << 32) | w1.x,
                                     ((unsigned long long)w1.w << 32) | w1.z};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (v[j] == key) return -2;
        if (v[j] == ~0ull) return j;
    }
    return -1;
}

__device__ __forceinline__ void gset_insert2(unsigned long long *tab, int64_t cap_mask,
                                             unsigned long long keyA, bool okA,
                                             unsigned long long keyB, bool okB, bool &newA,
                                             bool &newB, bool &full) {
    const uint64_t bA = okA ? gset_bucket(cap_mask, keyA) : 0, bB = okB ? gset_bucket(cap_mask, keyB) : 0;
    const uint4 *pA = reinterpret_cast<const uint4 *>(tab + bA);
    const uint4 *pB = reinterpret_cast<const uint4 *>(tab + bB);
    const uint4 a0 = pA[0], a1 = pA[1], b0 = pB[0], b1 = pB[1];
    const int sA = okA ? gset_scan4(a0, a1, keyA) : -2;
    const int sB = okB ? gset_scan4(b0, b1, keyB) : -2;
    unsigned long long oA = 0, oB = 0;
    if (sA >= 0) oA = atomicCAS(&tab[bA + sA], ~0ull, keyA);
    if (sB >= 0) oB = atomicCAS(&tab[bB + sB], ~0ull, keyB);
    newA = false;
    newB = false;
    if (okA && sA != -2) {
        if (sA >= 0 && oA == ~0ull) newA = true;
        else if (!(sA >= 0 && oA == keyA)) newA = gset_insert(tab, cap_mask, keyA, full);
    }
    if (okB && sB != -2) {
        if (sB >= 0 && oB == ~0ull) newB = true;
        else if (!(sB >= 0 && oB == keyB)) newB = gset_insert(tab, cap_mask, keyB, full);
    }
}

// The (task, id) set of the greedy phase.  Tasks below bm_tasks own a
// bitmap of n bits: membership is one atomic OR on a word of a contiguous
// per-task region (a task's probes stay within n/8 bytes, which caches
// well); later tasks fall back to the hash table.

// wave-wide: clear task t's bitmap (all lanes call this; a no-op for tasks
// that use the hash table).  The set is first updated by the greedy kernel,
// so the kernel boundary orders these stores before those updates and the
// wave does not wait for them.
__device__ __forceinline__ void tset_clear(const SearchBufs &sb, int64_t t) {
    if (t >= sb.bm_tasks) return;
    uint4 *p = reinterpret_cast<uint4 *>(sb.bm + t * sb.bm_words);
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    for (int64_t i = lane_id(); i < sb.bm_words / 4; i += 64) p[i] = z;
}

// add (t, id) to the set (seeds: known not to be present)
__device__ __forceinline__ void tset_add(const SearchBufs &sb, int64_t hmask, int64_t t, uint32_t id,
                                         bool &full) {
    if (t < sb.bm_tasks)
        atomicOr(&sb.bm[t * sb.bm_words + (id >> 5)], 1u << (id & 31));
    else
        gset_insert(sb.hash, hmask, ((unsigned long long)t << 32) | id, full);
}

// Logical block index that gives each XCD a contiguous share of the grid:
// the dispatcher deals workgroups to the 8 XCDs in turn, so consecutive
// logical blocks land on one XCD (and its L2) when the grid is a multiple
// of 8.
__device__ __forceinline__ int64_t xcd_block() {
    if (gridDim.x % 8 != 0) return blockIdx.x;
    return (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
}

// the value of lane (lane ^ J) for a compile-time J, in the VALU alone (no
// LDS round trip): DPP quad permutes for 1 and 2, a half-row mirror (lane ^ 7)
// and a quad reversal (lane ^ 3) for 4, a row rotation for 8, and the
// permlane swaps for 16 and 32 (odd rows of one copy trade places with even
// rows of another, or lanes 32-63 with lanes 0-31: the first copy's upper
// part then holds the lower part's values, the second copy's lower part the
// upper part's).  Every lane of the wave must be active.
template <int J> __device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
    if constexpr (J == 1) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);
    } else if constexpr (J == 2) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, false);
    } else if constexpr (J == 4) {
        const int m = __builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, false);
        return (uint32_t)__builtin_amdgcn_mov_dpp(m, 0x1B, 0xF, 0xF, false);
    } else if constexpr (J == 8) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, false);
    } else if constexpr (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (lane_id() & 16) ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (lane_id() & 32) ? r[0] : r[1];
    }
}
template <int J, typename D> __device__ __forceinline__ D xor_lane_d(D v) {
    if constexpr (sizeof(D) == 4) {
        return __builtin_bit_cast(D, xor_lane<J>(__builtin_bit_cast(uint32_t, v)));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = xor_lane<J>((uint32_t)u), hi = xor_lane<J>((uint32_t)(u >> 32));
        return __builtin_bit_cast(D, ((uint64_t)hi << 32) | lo);
    }
}

// sum over aligned groups of G lanes (every lane of the wave active)
template <int G, typename T> __device__ __forceinline__ T group_sum(T v) {
    if constexpr (G >= 2) v += xor_lane_d<1>(v);
    if constexpr (G >= 4) v += xor_lane_d<2>(v);
    if constexpr (G >= 8) v += xor_lane_d<4>(v);
    if constexpr (G >= 16) v += xor_lane_d<8>(v);
    if constexpr (G >= 32) v += xor_lane_d<16>(v);
    if constexpr (G >= 64) v += xor_lane_d<32>(v);
    return v;
}

// v[0, N): partial sums of N rounds held by every lane of a group of G.
// Exchanges at distances J, 2J, ... up to G/2: while a lane holds several
// rounds it keeps one half (the lower for a clear lane bit) and adds what the
// other lane held of it; v[0] ends as the group's sum of one round.
template <int J, int N, int G, typename T> __device__ __forceinline__ void scatter_sum(T *v, int lane) {
    if constexpr (J < G) {
        if constexpr (N > 1) {
            const bool up = (lane & J) != 0;
#pragma unroll
            for (int i = 0; i < N / 2; ++i) {
                const T keep = up ? v[i + N / 2] : v[i], send = up ? v[i] : v[i + N / 2];
                v[i] = keep + xor_lane_d<J>(send);
            }
            scatter_sum<2 * J, N / 2, G>(v, lane);
        } else {
            v[0] += xor_lane_d<J>(v[0]);
            scatter_sum<2 * J, 1, G>(v, lane);
        }
    }
}

// one compare-exchange stage of the bitonic network (merge size K, distance J)
template <int K, int J, typename D>
__device__ __forceinline__ void bitonic_stage(D &d, uint32_t &id, int lane) {
    const D od = xor_lane_d<J>(d);
    const uint32_t oi = xor_lane<J>(id);
    const bool up = (lane & K) == 0;
    const bool lower = (lane & J) == 0;
    bool take;
    if constexpr (sizeof(D) == 4 && D(-1) > D(0)) {
        // unsigned 32-bit distance: the (d, id) order is the order of the
        // 64-bit key d:id.  A lane keeps the smaller key when lower == up and
        // the larger one otherwise; for equal keys either choice leaves the
        // lane's value unchanged.
        const uint64_t mk = ((uint64_t)d << 32) | id, ok = ((uint64_t)od << 32) | oi;
        take = (ok < mk) != (lower != up);
    } else {
        take = (lower == up) ? key_less(od, oi, d, id) : key_less(d, id, od, oi);
    }
    if (take) {
        d = od;
        id = oi;
    }
}

// bitonic sort of one (d, id) pair per lane, ascending over lanes 0..63
// (called with every lane of the wave active)
template <typename D> __device__ __forceinline__ void wave_sort(D &d, uint32_t &id) {
    const int lane = lane_id();
    bitonic_stage<2, 1>(d, id, lane);
    bitonic_stage<4, 2>(d, id, lane);
    bitonic_stage<4, 1>(d, id, lane);
    bitonic_stage<8, 4>(d, id, lane);
    bitonic_stage<8, 2>(d, id, lane);
    bitonic_stage<8, 1>(d, id, lane);
    bitonic_stage<16, 8>(d, id, lane);
    bitonic_stage<16, 4>(d, id, lane);
    bitonic_stage<16, 2>(d, id, lane);
    bitonic_stage<16, 1>(d, id, lane);
    bitonic_stage<32, 16>(d, id, lane);
    bitonic_stage<32, 8>(d, id, lane);
    bitonic_stage<32, 4>(d, id, lane);
    bitonic_stage<32, 2>(d, id, lane);
    bitonic_stage<32, 1>(d, id, lane);
    bitonic_stage<64, 32>(d, id, lane);
    bitonic_stage<64, 16>(d, id, lane);
    bitonic_stage<64, 8>(d, id, lane);
    bitonic_stage<64, 4>(d, id, lane);
    bitonic_stage<64, 2>(d, id, lane);
    bitonic_stage<64, 1>(d, id, lane);
}

// --------------------------------------------------------------------------
// distance of a row chunk against the query chunk held in registers
// --------------------------------------------------------------------------

// Internal data type of the approximate pass on float data: rows are the
// bfloat16 copy, the query stays float32, squares accumulate in float32.
constexpr int RR_BF16X = 3;
// Internal data type of the 8-bit scalar-quantized pass: rows are codes,
// the query is float32 (prepared for the codes), sums accumulate in float32.
constexpr int RR_SQ8X = 4;
// Kernel data type = element type (low bits) | RR_IPBIT for the negated
// inner product (Section 2), so both metrics share every kernel template.
constexpr int RR_IPBIT = 8;
__host__ __device__ constexpr int dbase(int dt) { return dt & 7; }
__host__ __device__ constexpr bool dip(int dt) { return (dt & RR_IPBIT) != 0; }
// an approximate pass whose candidates are re-decided on the float32 rows
__host__ __device__ constexpr bool dapprox(int dt) { return dbase(dt) == RR_BF16X || dbase(dt) == RR_SQ8X; }
__host__ __device__ constexpr bool dfloat(int dt) { return dbase(dt) == RR_F32 || dapprox(dt); }
constexpr int RR_U8IP = RR_U8 | RR_IPBIT, RR_I8IP = RR_I8 | RR_IPBIT, RR_F32IP = RR_F32 | RR_IPBIT,
              RR_BF16XIP = RR_BF16X | RR_IPBIT, RR_SQ8XIP = RR_SQ8X | RR_IPBIT;

// T: the search key; Acc: the accumulator; O: the distance that decides
// membership and is reported (exact for every type).  Integer keys are
// unsigned: the inner product is searched as key_off - <p, q> >= 0.
template <int BASE> struct DistBase;
template <> struct DistBase<RR_U8> { using T = uint32_t; using Acc = int; using O = uint32_t; };
template <> struct DistBase<RR_I8> { using T = uint32_t; using Acc = int; using O = uint32_t; };
template <> struct DistBase<RR_F32> { using T = double; using Acc = double; using O = double; };
template <> struct DistBase<RR_BF16X> { using T = float; using Acc = float; using O = double; };
template <> struct DistBase<RR_SQ8X> { using T = float; using Acc = float; using O = double; };
template <int DTYPE> struct DistOf : DistBase<dbase(DTYPE)> {};

template <int DTYPE>
__device__ __forceinline__ typename DistOf<DTYPE>::Acc chunk_part(uint4 p, uint4 q);

// uint8: |p|^2 - 2 p.q over 16 bytes (|q|^2 is added once per row)
template <> __device__ __forceinline__ int chunk_part<RR_U8>(uint4 p, uint4 q) {
    unsigned pp = __builtin_amdgcn_udot4(p.x, p.x, 0u, false);
    pp = __builtin_amdgcn_udot4(p.y, p.y, pp, false);
    pp = __builtin_amdgcn_udot4(p.z, p.z, pp, false);
    pp = __builtin_amdgcn_udot4(p.w, p.w, pp, false);
    unsigned pq = __builtin_amdgcn_udot4(p.x, q.x, 0u, false);
    pq = __builtin_amdgcn_udot4(p.y, q.y, pq, false);
    pq = __builtin_amdgcn_udot4(p.z, q.z, pq, false);
    pq = __builtin_amdgcn_udot4(p.w, q.w, pq, false);
    return (int)pp - 2 * (int)pq;
}

template <> __device__ __forceinline__ int chunk_part<RR_I8>(uint4 p, uint4 q) {
    int pp = __builtin_amdgcn_sdot4((int)p.x, (int)p.x, 0, false);
    pp = __builtin_amdgcn_sdot4((int)p.y, (int)p.y, pp, false);
    pp = __builtin_amdgcn_sdot4((int)p.z, (int)p.z, pp, false);
    pp = __builtin_amdgcn_sdot4((int)p.w, (int)p.w, pp, false);
    int pq = __builtin_amdgcn_sdot4((int)p.x, (int)q.x, 0, false);
    pq = __builtin_amdgcn_sdot4((int)p.y, (int)q.y, pq, false);
    pq = __builtin_amdgcn_sdot4((int)p.z, (int)q.z, pq, false);
    pq = __builtin_amdgcn_sdot4((int)p.w, (int)q.w, pq, false);
    return pp - 2 * pq;
}

template <> __device__ __forceinline__ double chunk_part<RR_F32>(uint4 p, uint4 q) {
    double t0 = (double)__uint_as_float(p.x) - (double)__uint_as_float(q.x);
    double t1 = (double)__uint_as_float(p.y) - (double)__uint_as_float(q.y);
    double t2 = (double)__uint_as_float(p.z) - (double)__uint_as_float(q.z);
    double t3 = (double)__uint_as_float(p.w) - (double)__uint_as_float(q.w);
    double a = t0 * t0;
    a = fma(t1, t1, a);
    a = fma(t2, t2, a);
    a = fma(t3, t3, a);
    return a;
}

// inner-product parts: <p, q> over the chunk (uint8/int8: exact int32)
template <int BASE>
__device__ __forceinline__ typename DistBase<BASE>::Acc chunk_ip(uint4 p, uint4 q);
template <> __device__ __forceinline__ int chunk_ip<RR_U8>(uint4 p, uint4 q) {
    unsigned pq = __builtin_amdgcn_udot4(p.x, q.x, 0u, false);
    pq = __builtin_amdgcn_udot4(p.y, q.y, pq, false);
    pq = __builtin_amdgcn_udot4(p.z, q.z, pq, false);
    pq = __builtin_amdgcn_udot4(p.w, q.w, pq, false);
    return (int)pq;
}
template <> __device__ __forceinline__ int chunk_ip<RR_I8>(uint4 p, uint4 q) {
    int pq = __builtin_amdgcn_sdot4((int)p.x, (int)q.x, 0, false);
    pq = __builtin_amdgcn_sdot4((int)p.y, (int)q.y, pq, false);
    pq = __builtin_amdgcn_sdot4((int)p.z, (int)q.z, pq, false);
    pq = __builtin_amdgcn_sdot4((int)p.w, (int)q.w, pq, false);
    return pq;
}
template <> __device__ __forceinline__ double chunk_ip<RR_F32>(uint4 p, uint4 q) {
    double a = (double)__uint_as_float(p.x) * (double)__uint_as_float(q.x);
    a = fma((double)__uint_as_float(p.y), (double)__uint_as_float(q.y), a);
    a = fma((double)__uint_as_float(p.z), (double)__uint_as_float(q.z), a);
    a = fma((double)__uint_as_float(p.w), (double)__uint_as_float(q.w), a);
    return a;
}

// bfloat16 row chunk (8 values) against 8 float32 query values: sum of
// squared differences, float32 accumulation
__device__ __forceinline__ float chunk_part_bf16(uint4 p, uint4 q0, uint4 q1) {
    const uint32_t w[4] = {p.x, p.y, p.z, p.w};
    const uint32_t qa[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
    float a = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float lo = __uint_as_float(w[j] << 16);
        const float hi = __uint_as_float(w[j] & 0xffff0000u);
        const float t0 = lo - __uint_as_float(qa[2 * j]);
        const float t1 = hi - __uint_as_float(qa[2 * j + 1]);
        a = fmaf(t0, t0, a);
        a = fmaf(t1, t1, a);
    }
    return a;
}

// the same for the inner product: sum of products, float32 accumulation
__device__ __forceinline__ float chunk_ip_bf16(uint4 p, uint4 q0, uint4 q1) {
    const uint32_t w[4] = {p.x, p.y, p.z, p.w};
    const uint32_t qa[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
    float a = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        a = fmaf(__uint_as_float(w[j] << 16), __uint_as_float(qa[2 * j]), a);
        a = fmaf(__uint_as_float(w[j] & 0xffff0000u), __uint_as_float(qa[2 * j + 1]), a);
    }
    return a;
}

// 8-bit code chunk (16 codes) against 16 float32 query values prepared for
// the codes (q' = (q - lo) / scale): sum of squared differences in code
// units, float32 accumulation; the caller scales by scale^2
__device__ __forceinline__ float chunk_part_sq8(uint4 p, const uint4 *qc) {
    const uint32_t w[4] = {p.x, p.y, p.z, p.w};
    float a = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint4 q = qc[j];
        const float qa[4] = {__uint_as_float(q.x), __uint_as_float(q.y), __uint_as_float(q.z),
                             __uint_as_float(q.w)};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float t = (float)((w[j] >> (8 * k)) & 0xffu) - qa[k];
            a = fmaf(t, t, a);
        }
    }
    return a;
}

// the same for the inner product: sum of code * q (the caller scales by
// -scale; the lo <q, 1> part is a per-query constant kept in the thresholds)
__device__ __forceinline__ float chunk_ip_sq8(uint4 p, const uint4 *qc) {
    const uint32_t w[4] = {p.x, p.y, p.z, p.w};
    float a = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint4 q = qc[j];
        const float qa[4] = {__uint_as_float(q.x), __uint_as_float(q.y), __uint_as_float(q.z),
                             __uint_as_float(q.w)};
#pragma unroll
        for (int k = 0; k < 4; ++k) a = fmaf((float)((w[j] >> (8 * k)) & 0xffu), qa[k], a);
    }
    return a;
}

// |q|^2 part for integer data (float data needs none)
template <int DTYPE> __device__ __forceinline__ int chunk_qq(uint4 q);
template <> __device__ __forceinline__ int chunk_qq<RR_U8>(uint4 q) {
    unsigned s = __builtin_amdgcn_udot4(q.x, q.x, 0u, false);
    s = __builtin_amdgcn_udot4(q.y, q.y, s, false);
    s = __builtin_amdgcn_udot4(q.z, q.z, s, false);
    s = __builtin_amdgcn_udot4(q.w, q.w, s, false);
    return (int)s;
}
template <> __device__ __forceinline__ int chunk_qq<RR_I8>(uint4 q) {
    int s = __builtin_amdgcn_sdot4((int)q.x, (int)q.x, 0, false);
    s = __builtin_amdgcn_sdot4((int)q.y, (int)q.y, s, false);
    s = __builtin_amdgcn_sdot4((int)q.z, (int)q.z, s, false);
    s = __builtin_amdgcn_sdot4((int)q.w, (int)q.w, s, false);
    return s;
}

// Query state held by each lane: its CPL chunks of the padded query row.
// For the bfloat16 pass each 16-byte row chunk (8 values) pairs with 32
// bytes of the float32 query, so a lane holds 2*CPL query chunks.
// For the 8-bit pass each 16-byte chunk (16 codes) pairs with 64 bytes of
// float32 query, so a lane holds 4*CPL query chunks; the float32 query for
// the re-decision follows the prepared one in the query row.
template <int DTYPE, int CPL, int G> struct QueryRegs {
    static constexpr int QC = dbase(DTYPE) == RR_BF16X ? 2 * CPL : dbase(DTYPE) == RR_SQ8X ? 4 * CPL : CPL;
    static constexpr bool L2INT = !dfloat(DTYPE) && !dip(DTYPE);
    uint4 c[QC];
    int qq; // integer data: |q|^2 (L2) or the key offset (inner product)
    float sc; // 8-bit pass: scale^2 (L2) or -scale (inner product)
    const uint8_t *row; // the padded float32 query row (the recheck reads it)

    __device__ __forceinline__ void load(const uint8_t *qrow, const DevIndex &ix) {
        const int gl = lane_id() & (G - 1);
        row = dbase(DTYPE) == RR_SQ8X ? qrow + 4 * (size_t)ix.row_bytes : qrow;
        sc = dip(DTYPE) ? -ix.sq_scale : ix.sq_scale * ix.sq_scale;
        int s = 0;
#pragma unroll
        for (int k = 0; k < QC; ++k) {
            c[k] = *reinterpret_cast<const uint4 *>(qrow + (size_t)(gl * QC + k) * 16);
            if constexpr (L2INT) s += chunk_qq<dbase(DTYPE)>(c[k]);
        }
        if constexpr (L2INT) qq = group_sum<G>(s);
        else qq = (int)(uint32_t)ix.key_off;
    }
};

// Evaluate up to 64 candidates ci[0, k) (ids in LDS), one per lane: returns
// the distance of candidate `c` of this lane (meaningless where c >= k).  Row
// r of a batch of RB rounds is read by lane group r % (64/G); the sums over a
// group's lanes are reduced and scattered at once: at each exchange distance a
// lane passes on half of its rounds and keeps the other half, so RB rounds
// take RB - 1 exchanges instead of RB log2(RB), and every lane ends with one
// round's sum.  The additions pair the same lanes in the same order as
// group_sum.  8 to 12 chunk loads of a lane are in flight.
template <int DTYPE, int CPL, int G>
__device__ __forceinline__ typename DistOf<DTYPE>::T eval64(const DevIndex &ix, const QueryRegs<DTYPE, CPL, G> &qr,
                                                            const uint32_t *ci, int k, int &c) {
    using D = typename DistOf<DTYPE>::T;
    using Acc = typename DistOf<DTYPE>::Acc;
    constexpr int RPR = 64 / G; // rows per round
    constexpr int RBX = CPL == 1 ? 8 : CPL <= 3 ? 4 : 2;
    constexpr int RB = RBX < G ? RBX : G, NB = G / RB; // rounds per batch, batches
    const int lane = lane_id();
    const int gl = lane & (G - 1);
    const int grp = lane / G;
    Acc out = 0;
    const int mysel = (lane / RB) & (NB - 1);
#pragma unroll
    for (int bt = 0; bt < NB; ++bt) {
        if (bt * RB * RPR >= k) break;
        // every lane loads (past the end, the last candidate's row again): all
        // ids are read before the first load, and no load waits on a branch
        const uint8_t *row[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            const uint32_t id = ci[min((bt * RB + r) * RPR + grp, k - 1)];
            row[r] = ix.base + (uint64_t)id * (uint32_t)ix.row_bytes + gl * CPL * 16;
        }
        uint4 buf[RB][CPL];
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int kk = 0; kk < CPL; ++kk) buf[r][kk] = *reinterpret_cast<const uint4 *>(row[r] + kk * 16);
        Acc v[RB];
#pragma unroll
        for (int r = 0; r < RB; ++r) {
            Acc a = 0;
#pragma unroll
            for (int kk = 0; kk < CPL; ++kk) {
                if constexpr (DTYPE == RR_BF16X)
                    a += chunk_part_bf16(buf[r][kk], qr.c[2 * kk], qr.c[2 * kk + 1]);
                else if constexpr (DTYPE == RR_BF16XIP)
                    a += chunk_ip_bf16(buf[r][kk], qr.c[2 * kk], qr.c[2 * kk + 1]);
                else if constexpr (DTYPE == RR_SQ8X)
                    a += chunk_part_sq8(buf[r][kk], &qr.c[4 * kk]);
                else if constexpr (DTYPE == RR_SQ8XIP)
                    a += chunk_ip_sq8(buf[r][kk], &qr.c[4 * kk]);
                else if constexpr (dip(DTYPE))
                    a += chunk_ip<dbase(DTYPE)>(buf[r][kk], qr.c[kk]);
                else
                    a += chunk_part<DTYPE>(buf[r][kk], qr.c[kk]);
            }
            v[r] = a;
        }
        scatter_sum<1, RB, G>(v, lane);
        out = mysel == bt ? v[0] : out;
    }
    // the round a lane ended with: bit s of the lane chose the half of RB >> s
    int r = 0;
#pragma unroll
    for (int s = 0; (RB >> s) > 1; ++s) r += ((lane >> s) & 1) * (RB >> (s + 1));
    c = (mysel * RB + r) * RPR + grp;
    if constexpr (dbase(DTYPE) == RR_SQ8X) return (D)(out * qr.sc);
    else if constexpr (dfloat(DTYPE)) return (D)(dip(DTYPE) ? -out : out);
    else if constexpr (dip(DTYPE)) return (D)((uint32_t)qr.qq - (uint32_t)out);
    else return (D)(uint32_t)(out + qr.qq);
}

// FP64 distances of up to 64 points ci[0, k) (ids in LDS) from their float32
// rows, one per lane (meaningless from lane k on), for the approximate
// passes' decisions.  Rows are read and summed as the float32 search reads
// and sums them (lane groups, the same order), four rounds in flight.  One
// lane a row, 64 different lines per load, took 37 us for a level of the
// greedy phase on 768 values, however few points it held.
template <bool IP>
__device__ double exact64(const DevIndex &ix, const uint8_t *qrow, const uint32_t *ci, int k) {
    const int chunks = ix.row_bytes_exact / 16;
    const bool p2 = (chunks & (chunks - 1)) == 0;
    const int g = p2 ? min(chunks, 64) : min(chunks / 3, 64), cpl = chunks / g; // row_split
    const int lane = lane_id(), gl = lane & (g - 1), grp = lane / g, per = 64 / g;
    const uint4 *q = reinterpret_cast<const uint4 *>(qrow) + gl * cpl;
    double out = 0.0;
    for (int r0 = 0; r0 * per < k; r0 += 4) {
        const uint4 *x[4];
        double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t id = ci[min((r0 + r) * per + grp, k - 1)];
            x[r] = reinterpret_cast<const uint4 *>(ix.base_exact + (uint64_t)id * (uint32_t)ix.row_bytes_exact) + gl * cpl;
        }
        for (int kk = 0; kk < cpl; ++kk) {
            const uint4 y = q[kk];
            uint4 v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = x[r][kk];
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] += IP ? chunk_ip<RR_F32>(v[r], y) : chunk_part<RR_F32>(v[r], y);
        }
        for (int o = 1; o < g; o <<= 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) s[r] += __shfl_xor(s[r], o);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const double v = __shfl(s[r], (lane & (per - 1)) * g);
            out = lane / per == r0 + r ? v : out;
        }
    }
    return IP ? -out : out;
}

// in-range test and early-stop tests on the exact distance
template <typename D> __device__ __forceinline__ bool in_range(D d, const QThresh &t);
template <> __device__ __forceinline__ bool in_range<uint32_t>(uint32_t d, const QThresh &t) {
    return (int64_t)d <= t.r_int;
}
template <> __device__ __forceinline__ bool in_range<double>(double d, const QThresh &t) {
    return d <= t.r;
}
// approximate pass: used only by the early-stop test (membership is decided
// on the exact distance)
template <> __device__ __forceinline__ bool in_range<float>(float d, const QThresh &t) {
    return d <= t.r_f;
}
template <typename D> __device__ __forceinline__ bool beyond_esr(D d, const QThresh &t);
template <> __device__ __forceinline__ bool beyond_esr<uint32_t>(uint32_t d, const QThresh &t) {
    return (int64_t)d > t.esr_int;
}
template <> __device__ __forceinline__ bool beyond_esr<double>(double d, const QThresh &t) {
    return d > t.esr;
}
template <> __device__ __forceinline__ bool beyond_esr<float>(float d, const QThresh &t) {
    return d > t.esr_f;
}

// the kernels' data type: the index dtype, or the bfloat16 pass, with the
// metric bit
static inline int kernel_dtype(const DevIndex &ix, const SearchCfg &cfg) {
    int b = ix.dtype;
    if (ix.dtype == RR_F32 && cfg.precision == RR_BF16_RECHECK) b = RR_BF16X;
    if (ix.dtype == RR_F32 && cfg.precision == RR_SQ8_RERANK) b = RR_SQ8X;
    return b | (ix.metric == RR_IP ? RR_IPBIT : 0);
}

// stride of the padded query rows: the bfloat16 pass keeps float32 queries
// next to bf16 rows (twice the row stride); the 8-bit pass keeps the query
// prepared for the codes and the float32 query (4 + 4 times the stride)
template <int DTYPE> __device__ __forceinline__ size_t qrow_stride(const DevIndex &ix) {
    return dbase(DTYPE) == RR_BF16X ? 2 * (size_t)ix.row_bytes
           : dbase(DTYPE) == RR_SQ8X ? 8 * (size_t)ix.row_bytes
                                     : (size_t)ix.row_bytes;
}

// --------------------------------------------------------------------------
// the beam of one wave
// --------------------------------------------------------------------------

// Beam keys: the (d, id) order as unsigned integers.  The distance is mapped
// to an unsigned image in its order (-0 as +0, NaN last), the id is shifted
// left by one, and bit 0 says whether the point was visited (two keys of one
// beam never differ in that bit alone).  All ones is the empty key: it is
// after every other and counts as visited.
__device__ __forceinline__ uint32_t key_image(uint32_t d) { return d; }
__device__ __forceinline__ uint32_t key_image(float d) {
    const uint32_t b = __float_as_uint(d + 0.f);
    return d == d ? ((b >> 31) ? ~b : (b | 0x80000000u)) : 0xffffffffu;
}
__device__ __forceinline__ uint64_t key_image(double d) {
    const uint64_t b = (uint64_t)__double_as_longlong(d + 0.0);
    return d == d ? ((b >> 63) ? ~b : (b | 0x8000000000000000ull)) : ~0ull;
}
template <typename D> __device__ __forceinline__ D key_unimage(uint64_t k);
template <> __device__ __forceinline__ uint32_t key_unimage<uint32_t>(uint64_t k) { return (uint32_t)k; }
template <> __device__ __forceinline__ float key_unimage<float>(uint64_t k) {
    const uint32_t u = (uint32_t)k;
    return __uint_as_float((u >> 31) ? (u & 0x7fffffffu) : ~u);
}
template <> __device__ __forceinline__ double key_unimage<double>(uint64_t k) {
    return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}

__device__ __forceinline__ uint32_t read_lane(uint32_t v, int j) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, j);
}
// lane 0's value, known to be uniform
__device__ __forceinline__ int64_t uniform64(int64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// 32-bit distances: one 64-bit word.  FP64 distances: a 64-bit and a 32-bit word.
template <typename D> struct BeamKey {
    uint64_t v;
    static __device__ __forceinline__ BeamKey make(D d, uint32_t id) {
        return {((uint64_t)key_image(d) << 32) | (uint64_t)(id << 1)};
    }
    static __device__ __forceinline__ BeamKey empty() { return {~0ull}; }
    __device__ __forceinline__ bool less(const BeamKey &o) const { return v < o.v; }
    __device__ __forceinline__ bool same(const BeamKey &o) const { return (v | 1ull) == (o.v | 1ull); }
    __device__ __forceinline__ bool visited() const { return (v & 1ull) != 0; }
    __device__ __forceinline__ void visit() { v |= 1ull; }
    __device__ __forceinline__ bool is_empty() const { return v == ~0ull; }
    __device__ __forceinline__ uint32_t id() const { return (uint32_t)v >> 1; }
    __device__ __forceinline__ D dist() const { return key_unimage<D>(v >> 32); }
    __device__ __forceinline__ BeamKey lane(int j) const {
        return {((uint64_t)read_lane((uint32_t)(v >> 32), j) << 32) | read_lane((uint32_t)v, j)};
    }
    template <int J> __device__ __forceinline__ BeamKey xored() const {
        return {((uint64_t)xor_lane<J>((uint32_t)(v >> 32)) << 32) | xor_lane<J>((uint32_t)v)};
    }
};
template <> struct BeamKey<double> {
    uint64_t d;
    uint32_t i;
    static __device__ __forceinline__ BeamKey make(double x, uint32_t id) { return {key_image(x), id << 1}; }
    static __device__ __forceinline__ BeamKey empty() { return {~0ull, 0xffffffffu}; }
    __device__ __forceinline__ bool less(const BeamKey &o) const { return d < o.d || (d == o.d && i < o.i); }
    __device__ __forceinline__ bool same(const BeamKey &o) const { return d == o.d && (i | 1u) == (o.i | 1u); }
    __device__ __forceinline__ bool visited() const { return (i & 1u) != 0; }
    __device__ __forceinline__ void visit() { i |= 1u; }
    __device__ __forceinline__ bool is_empty() const { return d == ~0ull && i == 0xffffffffu; }
    __device__ __forceinline__ uint32_t id() const { return i >> 1; }
    __device__ __forceinline__ double dist() const { return key_unimage<double>(d); }
    __device__ __forceinline__ BeamKey lane(int j) const {
        return {((uint64_t)read_lane((uint32_t)(d >> 32), j) << 32) | read_lane((uint32_t)d, j), read_lane(i, j)};
    }
    template <int J> __device__ __forceinline__ BeamKey xored() const {
        return {((uint64_t)xor_lane<J>((uint32_t)(d >> 32)) << 32) | xor_lane<J>((uint32_t)d), xor_lane<J>(i)};
    }
};

// one compare-exchange stage: a lane keeps the smaller key where `lower` (its
// bit J clear) equals `up`
template <int J, typename K> __device__ __forceinline__ void key_stage(K &k, bool up, int lane) {
    const K o = k.template xored<J>();
    if (o.less(k) == (((lane & J) == 0) == up)) k = o;
}
template <int K0, int J, typename K> __device__ __forceinline__ void key_merge_steps(K &k, bool up, int lane) {
    key_stage<J>(k, up, lane);
    if constexpr (J > 1) key_merge_steps<K0, J / 2>(k, up, lane);
}
template <int S, typename K> __device__ __forceinline__ void key_sort_steps(K &k, bool up, int lane) {
    if constexpr (S > 2) key_sort_steps<S / 2>(k, up, lane);
    key_merge_steps<S, S / 2>(k, ((lane & S) == 0) == up, lane);
}

// Algorithm 1's beam B: the b best keys seen, visited or not.
//
// b <= 64: one key per lane, in order, empty keys above.  The ranks of new
// keys among the old ones and among themselves are population counts of one
// comparison each, and one trip through LDS puts every key in its lane; many
// at once are sorted and merged as two halves of a bitonic sequence.
//
// b > 64: a sorted array in LDS (`main`) plus up to 64 later keys in the
// lanes (`side`), which are merged into the array when they no longer fit
// the lanes: the array is moved once per about 64 insertions instead of at
// every visit.  Together they may hold more than b keys; a key whose rank
// among all of them is b or more is out of B, and stays out, because ranks
// only grow.  It is never handed out, and the merge drops it.  Once the seen
// cache has forgotten ids, new keys are looked up in main first (dropping the
// repeated ones only when they are merged or handed out was slower, 9.3 against
// 5.1 ms for 1,000 queries at b = 1,024: most of them are repeats by then).
//
// Both forms are about latency: a wave's visits form a chain, and the work
// between its two trips to memory is on it.  Beam kernel times when the beam
// was a sorted LDS array merged at every visit by binary searches, and now
// (1M x 128 uint8): 64 queries at b = 32 0.33 -> 0.16 ms; 10,000 at b = 8 0.34
// -> 0.22 ms; 1,000 at b = 1,024 8.5 -> 4.1 ms; doubling to 4,096 20 -> 5.9 ms.
template <typename D> struct WaveBeam {
    using K = BeamKey<D>;
    static constexpr bool WIDE_KEY = sizeof(D) == 8;
    uint64_t *mv; // main, in LDS: the keys, or the distances of FP64 keys
    uint32_t *mi; // FP64 keys: their second words
    uint64_t *xv; // scratch keys, laid out the same (first, the ids of a visit's candidates)
    uint32_t *xi;
    int b;
    K side;       // this lane's key
    int ns = 0;   // keys in the lanes
    int nM = 0;   // wide: keys in main
    K ck;         // wide: this lane's key of main's chunk at cbase (-1: none)
    int cbase = -1;
    int cursor = 0; // wide: main entries before it are visited
    int im = -1;  // wide: first unvisited entry of main (nM: none; -1: look)
    K km;         // its key
    K bound;      // keys not below it cannot enter

    __device__ __forceinline__ bool wide() const { return b > 64; }
    __device__ __forceinline__ K main_at(int i) const {
        if constexpr (WIDE_KEY) return K{mv[i], mi[i]};
        else return K{mv[i]};
    }
    __device__ __forceinline__ void main_set(int i, const K &k) {
        if constexpr (WIDE_KEY) {
            mv[i] = k.d;
            mi[i] = k.i;
        } else {
            mv[i] = k.v;
        }
    }
    __device__ __forceinline__ K scratch_at(int i) const {
        if constexpr (WIDE_KEY) return K{xv[i], xi[i]};
        else return K{xv[i]};
    }
    __device__ __forceinline__ void scratch_set(int i, const K &k) {
        if constexpr (WIDE_KEY) {
            xv[i] = k.d;
            xi[i] = k.i;
        } else {
            xv[i] = k.v;
        }
    }
    static __device__ __forceinline__ K pick(bool c, const K &a, const K &o) {
        K r;
        if constexpr (WIDE_KEY) {
            r.d = c ? a.d : o.d;
            r.i = c ? a.i : o.i;
        } else {
            r.v = c ? a.v : o.v;
        }
        return r;
    }

    // lds: wave_lds_bytes of bcap keys
    __device__ __forceinline__ void init(uint8_t *lds, int bcap, int width) {
        const int sk = beam_scratch_keys(bcap);
        xv = reinterpret_cast<uint64_t *>(lds);
        mv = xv + sk;
        xi = reinterpret_cast<uint32_t *>(mv + bcap);
        mi = xi + sk;
        reset(width);
    }
    __device__ __forceinline__ void reset(int width) {
        b = width;
        side = K::empty();
        bound = K::empty();
        ns = nM = cursor = 0;
        im = cbase = -1;
    }

    // B <- one key, held by a lane where `mine`
    __device__ __forceinline__ void start(const K &k, bool mine) {
        const K x = k.lane(__ffsll((long long)__ballot(mine)) - 1);
        if (lane_id() == 0) side = x;
        ns = 1;
        if (!wide()) bound = side.lane(b - 1);
    }

    // entries of main below k (per lane); three probes a round
    __device__ __forceinline__ int lower_bound(const K &k) const {
        int pos = 0, st = 1;
        while (4 * st <= nM) st *= 4;
        for (; st > 0; st >>= 2) {
            int c = 0;
#pragma unroll
            for (int j = 1; j <= 3; ++j) {
                const int i = pos + j * st - 1;
                const bool below = main_at(min(i, nM - 1)).less(k); // (read past no branch)
                c += (int)below & (int)(i < nM);
            }
            pos += c * st;
        }
        return pos;
    }

    // side into main.  Side key j ends at (main keys below it) + j; a bit
    // array of those places tells every other place which entry of main it
    // takes.  Places are filled from the top down, 256 at a time, all reads
    // before the writes: a place takes an entry at or below itself.
    __device__ void merge_side() {
        if (ns == 0) return;
        const int lane = lane_id();
        wave_sync();
        const int np = lane < ns ? lower_bound(side) + lane : 1 << 30;
        const int total = min(b, nM + ns), words = (total + 63) >> 6;
        for (int w = lane; w < words; w += 64) xv[w] = 0ull;
        wave_sync();
        if (np < total) atomicOr(reinterpret_cast<unsigned long long *>(xv + (np >> 6)), 1ull << (np & 63));
        wave_sync();
        const int first = __builtin_amdgcn_readfirstlane(np) >> 6; // places below it keep their keys
        for (int top = words - 1; top >= first; top -= 4) {
            K k[4];
            int to[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int w = top - j;
                to[j] = -1;
                if (w < first) continue;
                const uint64_t taken = xv[w];
                const int o = 64 * w + lane;
                const int before = __popcll(__ballot(np < 64 * w)) + mbcnt(taken);
                if (!((taken >> lane) & 1ull) && o < total) {
                    to[j] = o;
                    k[j] = main_at(o - before);
                }
            }
            wave_sync();
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (to[j] >= 0) main_set(to[j], k[j]);
            wave_sync();
        }
        if (np < total) main_set(np, side);
        // the first unvisited side key may now lie before the cursor
        const unsigned long long u = __ballot(np < total && !side.visited());
        if (u) cursor = min(cursor, (int)__builtin_amdgcn_readlane(np, __ffsll((long long)u) - 1));
        nM = total;
        ns = 0;
        im = cbase = -1;
        side = K::empty();
        wave_sync();
        if (nM == b) bound = main_at(b - 1).lane(0);
    }

    // the lanes of `t`, four at a time (one after the other, each step of the
    // loop would wait for the scalar unit): j is the lane (64: none left), x
    // its key (empty)
    template <typename F> static __device__ __forceinline__ void for_lanes(unsigned long long t, const K &c, F f) {
        while (t) {
            int j[4];
            K x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                j[i] = t ? __ffsll((long long)t) - 1 : 64;
                t &= t - 1; // 0 stays 0
                x[i] = pick(j[i] < 64, c.lane(j[i] & 63), K::empty());
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) f(j[i], x[i]);
        }
    }

    // add the lanes' new keys `c` where valid.  `dedupe`: keys of B may come
    // back (a cache forgot them) and are dropped; `repeats`: the lanes may
    // hold one key several times.
    __device__ void insert(K c, bool valid, bool dedupe, bool repeats = false) {
        const int lane = lane_id();
        unsigned long long m = __ballot(valid && c.less(bound));
        if (!m) return;
        if (dedupe && nM > 0) {
            bool again = false; // in main, visited or not
            if ((m >> lane) & 1ull) {
                const int lb = lower_bound(c);
                again = (int)main_at(min(lb, nM - 1)).same(c) & (int)(lb < nM);
            }
            m &= ~__ballot(again);
        }
        if (dedupe && (ns > 0 || repeats)) {
            const unsigned long long t = m;
            for_lanes(t, c, [&](int j, const K &x) {
                const unsigned long long bit = j < 64 ? 1ull << j : 0ull;
                if (__ballot(side.same(x))) m &= ~bit;
                else if (repeats && (m & bit)) m &= ~(__ballot(c.same(x)) & ~bit);
            });
        }
        if (wide() && ns + __popcll(m) > 64) {
            merge_side();
            m &= __ballot(c.less(bound));
        }
        const int k = __popcll(m);
        if (k == 0) return;
        c = pick((m >> lane) & 1ull, c, K::empty());
        const int total = wide() ? ns + k : min(b, ns + k);
        if (k > 24) {
            key_sort_steps<64>(c, false, lane);        // descending
            side = pick(c.less(side), c, side);        // the 64 smallest of both
            key_merge_steps<64, 32>(side, true, lane); // ascending
        } else {
            int np = 64, up = 0; // the new key's lane; the old key's way up
            for_lanes(m, c, [&](int j, const K &x) {
                const unsigned long long below = __ballot(side.less(x));
                const int pos = __popcll(below) + __popcll(__ballot(c.less(x)));
                np = lane == j ? pos : np;
                up += (below >> lane) & 1ull ? 0 : 1; // (the empty key moves no key)
            });
            wave_sync();
            if (lane < ns && lane + up < 64) scratch_set(lane + up, side);
            if (np < 64) scratch_set(np, c);
            wave_sync();
            side = scratch_at(lane);
            wave_sync();
        }
        ns = total;
        side = pick(lane < ns, side, K::empty());
        if (!wide()) bound = side.lane(b - 1);
    }

    // the smallest key of B
    __device__ __forceinline__ K best() const {
        const K s = side.lane(0);
        if (!wide() || nM == 0) return s;
        const K h = main_at(0).lane(0);
        return pick(s.less(h), s, h);
    }

    // p*: the first unvisited key of B.  Returns false if there is none.
    // `at`: its place, for visit(): a lane, or 64 + an entry of main.
    __device__ bool next(K &p, int &at) {
        const int lane = lane_id();
        const unsigned long long u = __ballot(!side.visited());
        const int js = u ? __ffsll((long long)u) - 1 : 0;
        if (!wide()) {
            if (!u) return false;
            p = side.lane(js);
            at = js;
            return true;
        }
        if (im < 0) {
            im = nM;
            for (int base = cursor & ~63; base < nM; base += 64) {
                const int i = base + lane;
                if (cbase != base) {
                    ck = i < nM ? main_at(i) : K::empty();
                    cbase = base;
                }
                const unsigned long long m = __ballot(i >= cursor && !ck.visited());
                if (m) {
                    const int j = __ffsll((long long)m) - 1;
                    im = base + j;
                    km = ck.lane(j);
                    break;
                }
            }
            cursor = im;
        }
        const bool has_m = im < nM;
        if (!has_m && !u) return false;
        const K ks = side.lane(js);
        const bool take_s = u && (!has_m || ks.less(km));
        // is the smaller one's rank below b?  (the keys before a key of rank
        // below b have ranks below b too)
        bool in_b = nM + ns <= b;
        if (!in_b && has_m) in_b = im + __popcll(__ballot(side.less(km))) < b;
        if (!in_b && take_s) {
            const int t = b - 1 - js; // js + (main keys below ks) < b
            in_b = t >= nM || !main_at(t).lane(0).less(ks);
        }
        if (!in_b) return false;
        p = pick(take_s, ks, km);
        at = take_s ? js : 64 + im;
        return true;
    }

    __device__ __forceinline__ void visit(int at) {
        const int lane = lane_id();
        if (at < 64) {
            if (lane == at) side.visit();
        } else {
            if (64 + cbase + lane == at) {
                ck.visit();
                main_set(at - 64, ck);
            }
            cursor = at - 64 + 1;
            im = -1;
        }
    }

    // B in order in main; returns its size
    __device__ int settle() {
        if (wide()) {
            merge_side();
            return nM;
        }
        const int lane = lane_id();
        wave_sync();
        if (lane < ns) main_set(lane, side);
        wave_sync();
        return ns;
    }

    // B from n stored keys (stored(i) for i < n, in order)
    template <typename F> __device__ void restore(int n, F stored) {
        const int lane = lane_id();
        if (!wide()) {
            side = lane < n ? stored(lane) : K::empty();
            ns = n;
            bound = side.lane(b - 1);
            return;
        }
        wave_sync();
        for (int i = lane; i < n; i += 64) main_set(i, stored(i));
        wave_sync();
        nM = n;
        if (nM == b) bound = main_at(b - 1).lane(0);
    }
};

// LDS bytes of a beam key: 32-bit distances in one word, FP64 ones in two
template <typename D> constexpr int32_t beam_key_bytes() { return sizeof(D) == 8 ? 12 : 8; }

// --------------------------------------------------------------------------
// beam kernel: Algorithm 1 (+ Algorithm 5), then Algorithm 6's decision
// --------------------------------------------------------------------------

struct BeamArgs {
    DevIndex ix;
    int64_t nq;
    SearchCfg cfg;
    SearchBufs sb;
    int32_t lds_per_wave;
    int32_t bcap;     // beam capacity in LDS
    // serving: work item k is query qlist[k]; state resumes/suspends B
    const int32_t *qlist;
    int64_t nwork;
    BeamState *state;
    void *st_d;       // [nq][bcap] keys of the stored beams
    uint32_t *st_i;   // [nq][bcap] ids (| visited bit)
    int32_t step_budget; // visits per call and query (0: run to the end)
    // early-stopping metrics at visit count probe_step (null: not recorded):
    // probe_m[q][4] = d_visited, d_top1, d_top10, d_start; probe_f[q][2] =
    // reached, found
    int32_t probe_step;
    double *probe_m;
    int8_t *probe_f;
};

// Waves per SIMD that the beam kernel's registers are held to: integer rows
// of up to 1 KB need about 120 registers, so four waves fit; the others hold
// more of a row at once (1M x 96 float32, 2,500 queries: 0.280 ms at three
// waves, 0.307 ms at two; at four they spill, 0.92 ms).
template <int DTYPE, int CPL> constexpr int beam_waves() { return !dfloat(DTYPE) && CPL == 1 ? 4 : 3; }

template <int DTYPE, int CPL, int G>
__global__ __launch_bounds__(512, (beam_waves<DTYPE, CPL>())) void k_beam(BeamArgs a) {
    using D = typename DistOf<DTYPE>::T;
    using O = typename DistOf<DTYPE>::O;
    using K = BeamKey<D>;
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t *my = smem + (size_t)wid * a.lds_per_wave;
    const int cs = a.cfg.cache_slots;
    const int cs_shift = 32 - (31 - __clz(cs >> 3));
    uint32_t *const ci = (uint32_t *)my; // the beam's scratch
    uint32_t *const htab = (uint32_t *)(my + a.lds_per_wave - 4 * cs);
    const DevIndex &ix = a.ix;
    const SearchCfg &cfg = a.cfg;
    const int R = ix.R;
    const int b = cfg.beam;
    WaveBeam<D> B;
    B.init(my, a.bcap, b);

    // The work queue is striped over QSTRIPES counters on separate lines (one
    // counter would serialize every fetch): stripe s hands out work items s,
    // s + QSTRIPES, s + 2 QSTRIPES, ...  A wave starts at its own stripe and
    // moves to the next one when a stripe runs dry; a stripe never refills, so
    // a wave that has passed every stripe is done.  A relaxed load skips
    // stripes already seen dry without an atomic.
    int stripe = __builtin_amdgcn_readfirstlane((int)(((int64_t)blockIdx.x * (blockDim.x >> 6) + wid) % QSTRIPES));
    int dry = 0;
    for (;;) {
        int32_t wk = -1; // (wave-uniform: held, like all that follows from it, in scalar registers)
        while (dry < QSTRIPES) {
            int32_t k = -1;
            if (lane == 0) {
                unsigned long long *c = &a.sb.counters[CTR_QSTRIPE + stripe * CTR_STRIDE];
                const unsigned long long seen =
                    __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((int64_t)stripe + (int64_t)seen * QSTRIPES < a.nwork) k = (int32_t)atomicAdd(c, 1ull);
            }
            k = __builtin_amdgcn_readfirstlane(k);
            if (k >= 0 && (int64_t)stripe + (int64_t)k * QSTRIPES < a.nwork) {
                wk = stripe + k * QSTRIPES;
                break;
            }
            stripe = stripe + 1 == QSTRIPES ? 0 : stripe + 1;
            ++dry;
        }
        if (wk < 0) break;
        const int64_t q = a.qlist ? __builtin_amdgcn_readfirstlane(a.qlist[wk]) : wk;

        const QThresh th = a.sb.qth[q];
        QueryRegs<DTYPE, CPL, G> qr;
        qr.load(a.sb.qpad + (size_t)q * qrow_stride<DTYPE>(ix), ix);

        for (int i = lane; i < cs / 4; i += 64)
            reinterpret_cast<uint4 *>(htab)[i] = make_uint4(RR_EMPTY32, RR_EMPTY32, RR_EMPTY32, RR_EMPTY32);
        wave_sync();

        bool ovf = false;
        bool dedupe = false; // the cache may have forgotten points of B
        int visits = 0, evals = 1;
        int edges = 0; // adjacency entries read by the visits (sum of out-degrees)
        bool es_fired = false;
        B.reset(b);
        if (a.state && (a.state[q].flags & BS_STARTED)) {
            // resume: B as it was stored; the visited cache starts empty,
            // which is exact because the cache may forget ids
            const BeamState bs = a.state[q];
            visits = __builtin_amdgcn_readfirstlane(bs.visits);
            evals = __builtin_amdgcn_readfirstlane(bs.evals);
            edges = __builtin_amdgcn_readfirstlane(bs.edges);
            ovf = lane == 0 && (bs.flags & BS_OVF);
            dedupe = true;
            const D *sd = (const D *)a.st_d + (size_t)q * a.bcap;
            const uint32_t *si = a.st_i + (size_t)q * a.bcap;
            B.restore(__builtin_amdgcn_readfirstlane(bs.nB), [&](int i) {
                K k = K::make(sd[i], si[i] & RR_IDMASK);
                if (si[i] & RR_VIS) k.visit();
                return k;
            });
        } else {
            // B <- S = {entry}
            if (lane == 0) {
                ci[0] = (uint32_t)ix.entry;
                seen_insert(htab, cs_shift, (uint32_t)ix.entry, ovf);
            }
            wave_sync();
            int c = 0;
            const D d0 = eval64<DTYPE, CPL, G>(ix, qr, ci, 1, c);
            B.start(K::make(d0, (uint32_t)ix.entry), c == 0);
            if (a.probe_m && c == 0) {
                const double nan = __builtin_nan("");
                a.probe_m[4 * q] = nan;
                a.probe_m[4 * q + 1] = nan;
                a.probe_m[4 * q + 2] = nan;
                a.probe_m[4 * q + 3] = (double)d0 - (double)ix.key_off;
                a.probe_f[2 * q] = 0;
                a.probe_f[2 * q + 1] = 0;
            }
        }
        int steps = 0;
        bool suspend = false;

        for (;;) {
            K p;
            int at;
            if (!B.next(p, at)) break;
            if (a.probe_m && visits == a.probe_step) {
                const int nB = B.settle();
                if (lane == 0) {
                    const double ko = (double)ix.key_off;
                    a.probe_m[4 * q] = (double)p.dist() - ko;
                    a.probe_m[4 * q + 1] = (double)B.main_at(0).dist() - ko;
                    a.probe_m[4 * q + 2] = nB >= 10 ? (double)B.main_at(9).dist() - ko : __builtin_inf();
                    a.probe_f[2 * q] = 1;
                    a.probe_f[2 * q + 1] = in_range<D>(B.main_at(0).dist(), th) ? 1 : 0;
                }
                B.next(p, at); // settling may have moved p*
            }
            // Algorithm 5: min_B d > r, v >= vl, d(p*) > esr
            if (cfg.es_enable && visits >= cfg.vl && !in_range<D>(B.best().dist(), th) &&
                beyond_esr<D>(p.dist(), th)) {
                es_fired = true;
                break;
            }
            if (a.step_budget > 0 && steps >= a.step_budget) {
                suspend = true; // p* stays unvisited; the next call picks it again
                break;
            }
            ++steps;
            // N_out(p*), drop ids already evaluated
            int32_t f = ix.adj[(uint64_t)p.id() * (uint32_t)R + max(0, min(lane, R - 1))];
            if (lane >= R) f = -1;
            B.visit(at);
            ++visits;
            edges += __popcll(__ballot(f >= 0));
            bool cand = false;
            if (f >= 0) cand = !seen_insert(htab, cs_shift, (uint32_t)f, ovf);
            const unsigned long long cm = __ballot(cand);
            const int k = __popcll(cm);
            if (k == 0) continue;
            if (cand) ci[mbcnt(cm)] = (uint32_t)f;
            wave_sync();
            evals += k;
            int c = 0;
            const D d = eval64<DTYPE, CPL, G>(ix, qr, ci, k, c);
            // a key of B can only come back once the cache has forgotten one
            dedupe = dedupe || __ballot(ovf) != 0ull;
            const uint32_t id = ci[min(c, 63)];
            wave_sync();
            B.insert(K::make(d, id), c < k, dedupe);
        }

        // B in order in LDS
        const int nB = B.settle();
        if (suspend) {
            D *sd = (D *)a.st_d + (size_t)q * a.bcap;
            uint32_t *si = a.st_i + (size_t)q * a.bcap;
            for (int i = lane; i < nB; i += 64) {
                const K k = B.main_at(i);
                sd[i] = k.dist();
                si[i] = k.id() | (k.visited() ? RR_VIS : 0u);
            }
            const bool any_ovf = __ballot(ovf) != 0ull;
            if (lane == 0) {
                BeamState bs;
                bs.nB = nB;
                bs.visits = visits;
                bs.evals = evals;
                bs.flags = BS_STARTED | (any_ovf ? BS_OVF : 0);
                bs.edges = edges;
                a.state[q] = bs;
            }
            wave_sync();
            continue;
        }
        if (a.state && lane == 0) a.state[q].flags = BS_STARTED | BS_DONE;
        // N = the in-range points of B.  Exact types: an in-range prefix of
        // the sorted beam.  Approximate pass: the prefix with s <= hi holds
        // every possible member; each is re-decided on its exact distance.
        int cN = 0, cH = 0, nband = 0;
        double dx0 = 0.0; // the first 64 candidates' exact distances
        // exact distance of candidate base + lane
        auto recheck = [&](int base) {
            wave_sync();
            ci[lane] = B.main_at(min(base + lane, nB - 1)).id();
            wave_sync();
            const double dx = exact64<dip(DTYPE)>(ix, qr.row, ci, min(64, cH - base));
            wave_sync();
            return dx;
        };
        if constexpr (dapprox(DTYPE)) {
            for (int base = 0; base < nB; base += 64) {
                const int i = base + lane;
                const int c = __popcll(__ballot(i < nB && B.main_at(i).dist() <= th.hi));
                cH += c;
                if (c < 64) break;
            }
            for (int base = 0; base < cH; base += 64) {
                const int i = base + lane;
                const double dx = recheck(base);
                if (base == 0) dx0 = dx;
                cN += __popcll(__ballot(i < cH && dx <= th.r));
                nband += __popcll(__ballot(i < cH && B.main_at(i).dist() > th.lo));
            }
        } else {
            for (int base = 0; base < nB; base += 64) {
                const int i = base + lane;
                const bool inr = i < nB && in_range<D>(B.main_at(i).dist(), th);
                const int c = __popcll(__ballot(inr));
                cN += c;
                if (c < 64) break;
            }
        }
        // Algorithm 6: expand iff |N| >= lambda b; an empty N expands to nothing
        const bool expand_flag = cfg.mode == RR_ADAPTIVE && cN >= cfg.expand_thresh;
        const bool expand = expand_flag && cN > 0;
        // results of the approximate pass are sorted by exact distance in the
        // finalisation, so every non-empty query becomes a task there
        const bool as_task = expand || (dapprox(DTYPE) && cN > 0);
        rr_query_stats st;
        st.visits = visits;
        st.evals = evals;
        st.edges = edges;
        st.greedy_edges = 0;
        st.greedy_visits = 0;
        st.greedy_evals = 0;
        st.count = as_task ? 0 : cN;
        st.final_beam = b;
        st.es_fired = es_fired ? 1 : 0;
        st.expanded = expand_flag ? 1 : 0;
        st.truncated = 0;
        st.cache_overflow = __ballot(ovf) ? 1 : 0;
        st.rechecked = nband;
        st.rounds = 1;
        if (!as_task && (int64_t)cN > a.sb.max_results) {
            // more than max_results_per_query: the nearest ones are returned
            st.truncated = 1;
            cN = (int)a.sb.max_results;
            st.count = cN;
        }
        if (!as_task) {
            int64_t off = 0;
            if (lane == 0 && cN > 0) off = (int64_t)atomicAdd(&a.sb.counters[CTR_ARENA], (unsigned long long)cN);
            off = uniform64(off);
            if (cN > 0 && off + cN > a.sb.arena_cap) {
                st.truncated = 1;
                st.count = 0;
                if (lane == 0) atomicOr(&a.sb.counters[CTR_OVERFLOW], 1ull);
            } else {
                O *ad = (O *)a.sb.arena_dists;
                for (int i = lane; i < cN; i += 64) {
                    a.sb.arena_ids[off + i] = (int32_t)B.main_at(i).id();
                    ad[off + i] = (O)B.main_at(i).dist();
                }
            }
            if (lane == 0) {
                a.sb.res_off[q] = off;
                a.sb.res_cnt[q] = st.count;
            }
        } else {
            // a task of the greedy phase: N goes to level 0 (expanded only if
            // `expand`; otherwise it is just sorted and emitted)
            int64_t t = 0;
            if (lane == 0) t = (int64_t)atomicAdd(&a.sb.counters[CTR_TASKS], 1ull);
            t = uniform64(t);
            // (the task-local kernel clears, or writes, the bitmaps it needs)
            if (expand && a.sb.local_grid == 0) tset_clear(a.sb, t);
            bool full = false;
            O *idist = (O *)a.sb.item_dist;
            int64_t off = 0;
            if (lane == 0)
                off = (int64_t)(atomicAdd(&a.sb.level_cnt[0], (unsigned long long)cN));
            off = uniform64(off);
            auto put = [&](int64_t o, uint32_t id, O d) {
                if (o >= a.sb.item_cap) {
                    full = true;
                    return;
                }
                a.sb.item_key[o] = ((unsigned long long)(uint32_t)t << 32) | id;
                idist[o] = d;
            };
            if constexpr (dapprox(DTYPE)) {
                int64_t o = off;
                for (int base = 0; base < cH; base += 64) {
                    const int i = base + lane;
                    const double dx = base == 0 ? dx0 : recheck(base);
                    const unsigned long long im = __ballot(i < cH && dx <= th.r);
                    if ((im >> lane) & 1ull) put(o + mbcnt(im), B.main_at(i).id(), dx);
                    o += __popcll(im);
                }
            } else {
                for (int i = lane; i < cN; i += 64) put(off + i, B.main_at(i).id(), (O)B.main_at(i).dist());
            }
            const int written = (int)max((int64_t)0, min((int64_t)cN, a.sb.item_cap - off));
            const bool lost = __ballot(full) != 0ull;
            if (lost) {
                st.truncated = 1;
                if (lane == 0) atomicOr(&a.sb.counters[CTR_OVERFLOW], 2ull);
            }
            if (lane == 0) {
                a.sb.task_trunc[t] = lost ? 1 : 0;
                a.sb.task_q[t] = (int32_t)q;
                a.sb.task_cnt[t] = (unsigned long long)written;
                a.sb.task_prev[t] = (unsigned long long)written;
                a.sb.task_evals[t] = 0ull;
                a.sb.task_rechk[t] = 0ull;
                a.sb.task_expand[t] = expand ? 1 : 0;
                a.sb.task_out[t] = off;
                a.sb.res_off[q] = 0;
                a.sb.res_cnt[q] = 0;
            }
        }
        if (lane == 0) a.sb.stats[q] = st;
        wave_sync();
    }
}

// --------------------------------------------------------------------------
// doubling search: Algorithm 3 (with Algorithm 5's stop in every round when
// enabled), one wavefront per query
// --------------------------------------------------------------------------

// Each round is Algorithm 1 with width b started from S, the set of points
// visited in earlier rounds (the entry in round 1).  The search ends when the
// round's in-range points number fewer than lambda * b; otherwise b doubles,
// and a round that ends at b >= max_beam marks the result truncated.  A beam
// started from all of S is trimmed to its b best keys right after its first
// visit, which takes S's best key, so starting from the b best keys of S
// gives the same beam; the visited-cache argument of the beam kernel then
// applies unchanged.  S is kept as the list of visits of every round, with
// repeats (a repeated point has the same key and is dropped when the list is
// merged into the beam), in a region of HBM owned by the wave.
template <typename T> __device__ __forceinline__ T load_l2(const T *p) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "4- or 8-byte values");
    using U = typename std::conditional<sizeof(T) == 4, uint32_t, unsigned long long>::type;
    const U u = __hip_atomic_load(reinterpret_cast<const U *>(p), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    T v;
    __builtin_memcpy(&v, &u, sizeof v);
    return v;
}

struct DoublingArgs {
    DevIndex ix;
    SearchCfg cfg;
    SearchBufs sb;
    int64_t nq;
    int32_t lds_per_wave;
    int32_t bcap;      // the widest beam a round can use
    uint8_t *s_pool;   // per wave: s_cap keys, then s_cap ids
    int64_t s_cap;
};

template <int DTYPE, int CPL, int G>
__global__ __launch_bounds__(512) void k_doubling(DoublingArgs a) {
    using D = typename DistOf<DTYPE>::T;
    using O = typename DistOf<DTYPE>::O;
    using K = BeamKey<D>;
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint8_t *my = smem + (size_t)wid * a.lds_per_wave;
    const int bcap = a.bcap;
    const int cs = a.cfg.cache_slots;
    const int cs_shift = 32 - (31 - __clz(cs >> 3));
    uint32_t *const ci = (uint32_t *)my; // the beam's scratch
    uint32_t *const htab = (uint32_t *)(my + a.lds_per_wave - 4 * cs);
    WaveBeam<D> B;
    B.init(my, bcap, a.cfg.beam);
    const DevIndex &ix = a.ix;
    const SearchCfg &cfg = a.cfg;
    const int R = ix.R;
    const int64_t gw = (int64_t)blockIdx.x * (blockDim.x >> 6) + wid;
    D *const sd = (D *)(a.s_pool + (size_t)gw * (size_t)a.s_cap * (sizeof(D) + 4));
    uint32_t *const si = (uint32_t *)(sd + a.s_cap);

    for (;;) {
        int32_t qi = 0; // at most nq + the number of waves
        if (lane == 0) qi = (int32_t)atomicAdd(&a.sb.counters[CTR_QUEUE], 1ull);
        const int64_t q = (int64_t)(uint32_t)__builtin_amdgcn_readfirstlane(qi);
        if (q >= a.nq) break;

        const QThresh th = a.sb.qth[q];
        QueryRegs<DTYPE, CPL, G> qr;
        qr.load(a.sb.qpad + (size_t)q * qrow_stride<DTYPE>(ix), ix);

        bool ovf = false, trunc = false, es_any = false;
        int b = cfg.beam, rounds = 0, cN = 0;
        int64_t ns = 0, visits_all = 0, evals_all = 0, edges_all = 0;

        for (;;) {
            for (int i = lane; i < cs / 4; i += 64)
                reinterpret_cast<uint4 *>(htab)[i] = make_uint4(RR_EMPTY32, RR_EMPTY32, RR_EMPTY32, RR_EMPTY32);
            wave_sync();
            B.reset(b);
            int evals = 0;
            // the cache starts empty: points of S come back as neighbours
            bool dedupe = rounds > 0;
            if (rounds == 0) {
                // B <- S = {entry}
                if (lane == 0) {
                    ci[0] = (uint32_t)ix.entry;
                    seen_insert(htab, cs_shift, (uint32_t)ix.entry, ovf);
                }
                wave_sync();
                int c = 0;
                const D d0 = eval64<DTYPE, CPL, G>(ix, qr, ci, 1, c);
                B.start(K::make(d0, (uint32_t)ix.entry), c == 0);
                evals = 1;
            } else {
                // B <- the b best keys of S.  S was written by lane 0; the
                // stores are completed, then read at L2 (agent-scope loads
                // bypass the per-CU cache, which may hold an older query's S)
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                for (int64_t c0 = 0; c0 < ns; c0 += 64) {
                    K k = K::empty();
                    if (c0 + lane < ns) k = K::make(load_l2(sd + c0 + lane), load_l2(si + c0 + lane));
                    B.insert(k, c0 + lane < ns, true, true);
                }
            }
            int visits = 0;
            bool es_fired = false;
            for (;;) {
                K p;
                int at;
                if (!B.next(p, at)) break;
                // Algorithm 5 within the round: min_B d > r, v >= vl, d(p*) > esr
                if (cfg.es_enable && visits >= cfg.vl && !in_range<D>(B.best().dist(), th) &&
                    beyond_esr<D>(p.dist(), th)) {
                    es_fired = true;
                    break;
                }
                int32_t f = ix.adj[(uint64_t)p.id() * (uint32_t)R + max(0, min(lane, R - 1))];
                if (lane >= R) f = -1;
                B.visit(at);
                ++visits;
                // S <- S u {p*}
                if (ns < a.s_cap) {
                    if (lane == 0) {
                        sd[ns] = p.dist();
                        si[ns] = p.id();
                    }
                    ++ns;
                } else {
                    trunc = true;
                }
                edges_all += __popcll(__ballot(f >= 0));
                bool cand = false;
                if (f >= 0) cand = !seen_insert(htab, cs_shift, (uint32_t)f, ovf);
                const unsigned long long cm = __ballot(cand);
                const int k = __popcll(cm);
                if (k == 0) continue;
                if (cand) ci[mbcnt(cm)] = (uint32_t)f;
                wave_sync();
                evals += k;
                int c = 0;
                const D d = eval64<DTYPE, CPL, G>(ix, qr, ci, k, c);
                dedupe = dedupe || __ballot(ovf) != 0ull;
                const uint32_t id = ci[min(c, 63)];
                wave_sync();
                B.insert(K::make(d, id), c < k, dedupe);
            }
            visits_all += visits;
            evals_all += evals;
            es_any = es_any || es_fired;
            ++rounds;
            cN = 0;
            const int nB = B.settle();
            for (int base = 0; base < nB; base += 64) {
                const int i = base + lane;
                const int c = __popcll(__ballot(i < nB && in_range<D>(B.main_at(i).dist(), th)));
                cN += c;
                if (c < 64) break;
            }
            if ((double)cN < cfg.lambda * (double)b) break;
            if ((int64_t)b >= cfg.max_beam || 2 * b > bcap) {
                trunc = true;
                break;
            }
            b *= 2;
        }

        rr_query_stats st;
        st.visits = (int32_t)min(visits_all, (int64_t)INT32_MAX);
        st.evals = (int32_t)min(evals_all, (int64_t)INT32_MAX);
        st.edges = (int32_t)min(edges_all, (int64_t)INT32_MAX);
        st.greedy_edges = 0;
        st.greedy_visits = 0;
        st.greedy_evals = 0;
        st.count = cN;
        st.final_beam = b;
        st.es_fired = es_any ? 1 : 0;
        st.expanded = 0;
        st.truncated = trunc ? 1 : 0;
        st.cache_overflow = __ballot(ovf) ? 1 : 0;
        st.rechecked = 0;
        st.rounds = rounds;
        if ((int64_t)cN > a.sb.max_results) {
            // more than max_results_per_query: the nearest ones are returned
            st.truncated = 1;
            cN = (int)a.sb.max_results;
            st.count = cN;
        }
        int64_t off = 0;
        if (lane == 0 && cN > 0) off = (int64_t)atomicAdd(&a.sb.counters[CTR_ARENA], (unsigned long long)cN);
        off = uniform64(off);
        if (cN > 0 && off + cN > a.sb.arena_cap) {
            st.truncated = 1;
            st.count = 0;
            if (lane == 0) atomicOr(&a.sb.counters[CTR_OVERFLOW], 1ull);
        } else {
            O *ad = (O *)a.sb.arena_dists;
            for (int i = lane; i < cN; i += 64) {
                a.sb.arena_ids[off + i] = (int32_t)B.main_at(i).id();
                ad[off + i] = (O)B.main_at(i).dist();
            }
        }
        if (lane == 0) {
            a.sb.res_off[q] = off;
            a.sb.res_cnt[q] = st.count;
            a.sb.stats[q] = st;
        }
        wave_sync();
    }
}

// In-range decision of up to 64 candidates ci[0, k) (ids in LDS), one per
// lane: `in` marks the lanes whose candidate `id`, at distance `d`, lies in
// the ball.  Approximate passes decide exactly every candidate at or below
// the band's upper edge (xi: 64 ids of scratch) and count those above its
// lower one.
template <int DTYPE, int CPL, int G>
__device__ __forceinline__ void decide64(const DevIndex &ix, const QueryRegs<DTYPE, CPL, G> &qr, const QThresh &th,
                                         const uint32_t *ci, int k, uint32_t *xi, typename DistOf<DTYPE>::O &d,
                                         uint32_t &id, bool &in, unsigned long long &band) {
    int c = 0;
    const auto s = eval64<DTYPE, CPL, G>(ix, qr, ci, k, c);
    id = ci[min(c, k - 1)];
    if constexpr (dapprox(DTYPE)) {
        const int lane = lane_id();
        const bool need = c < k && s <= th.hi;
        const unsigned long long m = __ballot(need);
        in = false;
        if (!m) return;
        band += (unsigned long long)__popcll(__ballot(need && s > th.lo));
        wave_sync();
        if (need) xi[mbcnt(m)] = id;
        wave_sync();
        const int n = __popcll(m);
        d = exact64<dip(DTYPE)>(ix, qr.row, xi, n);
        id = xi[min(lane, n - 1)];
        in = lane < n && d <= th.r;
        wave_sync();
    } else {
        d = s;
        in = c < k && in_range<typename DistOf<DTYPE>::T>(s, th);
    }
}

// --------------------------------------------------------------------------
// greedy phase: Algorithm 2 for all tasks at once, level-synchronous
// --------------------------------------------------------------------------

struct LocalBusy {
    int low, high; // of local_busy
};
struct GreedyArgs {
    DevIndex ix;
    SearchCfg cfg;
    SearchBufs sb;
    LocalBusy busy; // task-local kernel
};

// Work layout.  The items of one level are grouped by task: level 0 is
// written that way by the beam kernel, and each later level is regrouped
// once it is complete.  Every workgroup expands one contiguous block of a
// level, so its waves mostly expand points of the same task, and they share
// one LDS cache of the (task, id) keys they already sent to the global set.
// Neighbour ids repeat heavily inside a block (points of one ball share most
// of their neighbours), and the cache keeps those repeats away from the
// global hash table, whose random probes bound this kernel.
constexpr int GREEDY_CACHE = 8192;  // workgroup-shared LDS cache of (task, id) keys
constexpr int GREEDY_STAGE = 128;   // per-wave staged outputs before a global reservation
constexpr int GREEDY_QUEUE = 192;   // per-wave queue of candidates awaiting distances

// waves per workgroup (one workgroup per CU): 16, or 8 where the distance
// code needs more than the 128 registers a 1024-lane workgroup leaves
template <int DTYPE, int CPL> constexpr int greedy_waves() {
    return (dfloat(DTYPE) || CPL >= 6) ? 8 : 16;
}

template <typename D, typename O, int GW> struct GreedyLds {
    unsigned long long cache[GREEDY_CACHE];
    uint32_t ci[GW][GREEDY_QUEUE];
    uint32_t xi[GW][64]; // approximate passes: ids to decide exactly
    uint32_t st_id[GW][GREEDY_STAGE];
    int32_t st_task[GW][GREEDY_STAGE];
    O st_d[GW][GREEDY_STAGE];
    int32_t st_n[GW];
    unsigned long long wg_base;
    unsigned long long part[GW * 64]; // task-segment scan
};

// true if `key` was already in the workgroup cache; otherwise it is added
// (evicting another key if its probe window is full: the cache may forget)
__device__ __forceinline__ bool wg_cache_seen(unsigned long long *cache, unsigned long long key) {
    const uint32_t h = hash32((uint32_t)key ^ hash32((uint32_t)(key >> 32)));
#pragma unroll 1
    for (int p = 0; p < 8; ++p) {
        const uint32_t s = (h + (uint32_t)p) & (GREEDY_CACHE - 1);
        const unsigned long long v = cache[s];
        if (v == key) return true;
        if (v == ~0ull) {
            const unsigned long long old = atomicCAS(&cache[s], ~0ull, key);
            if (old == ~0ull) return false;
            if (old == key) return true;
        }
    }
    cache[h & (GREEDY_CACHE - 1)] = key;
    return false;
}

// write a wave's staged outputs to the unsorted next level [dst, dst + n);
// every slot below item_cap is written, so the regrouping never reads an
// unwritten item
template <typename D, typename O, int GW>
__device__ __forceinline__ void greedy_emit(GreedyLds<D, O, GW> &L, int wid, int n, int64_t dst,
                                            const SearchBufs &sb) {
    const int lane = lane_id();
    O *udist = (O *)sb.u_dist;
    for (int i = lane; i < n; i += 64) {
        const int64_t o = dst + i;
        if (o < sb.item_cap) {
            sb.u_key[o] = ((unsigned long long)(uint32_t)L.st_task[wid][i] << 32) | L.st_id[wid][i];
            udist[o] = L.st_d[wid][i];
        } else {
            sb.task_trunc[L.st_task[wid][i]] = 1; // the item is dropped
        }
    }
    // results per task, one atomic per run of equal tasks (runs are contiguous)
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int i = i0 + lane;
        const bool valid = i < n && dst + i < sb.item_cap;
        const int32_t t = valid ? L.st_task[wid][i] : -1;
        const int32_t tprev = __shfl_up(t, 1);
        const bool head = valid && (lane == 0 || tprev != t);
        const unsigned long long hm = __ballot(head);
        const unsigned long long vm = __ballot(valid);
        if (head) {
            // run length: up to the next head or the end of the valid lanes
            const unsigned long long later = hm & ~((2ull << lane) - 1ull);
            const int end = later ? __ffsll((long long)later) - 1 : 64 - __clzll((long long)vm);
            atomicAdd(&sb.task_cnt[t], (unsigned long long)(end - lane));
        }
    }
    if (dst + n > sb.item_cap && lane == 0) atomicOr(&sb.counters[CTR_OVERFLOW], 4ull);
}

// in-place inclusive scan of part[0, blockDim.x) by the whole workgroup
// (Hillis-Steele, log2(blockDim.x) barrier pairs)
static __device__ void block_inclusive_scan(unsigned long long *part) {
    const int tid = threadIdx.x;
    for (int off = 1; off < (int)blockDim.x; off <<= 1) {
        const unsigned long long v = tid >= off ? part[tid - off] : 0ull;
        __syncthreads();
        part[tid] += v;
        __syncthreads();
    }
}

// one workgroup: seg_off[t] = start of task t's items in the next level,
// from the per-task growth task_cnt - task_prev; resets the scatter cursors
static __device__ void greedy_segments(unsigned long long *part, const SearchBufs &sb, int64_t ntasks,
                                int64_t next_base) {
    const int tid = threadIdx.x;
    const int nth = blockDim.x;
    const int64_t per = (ntasks + nth - 1) / nth;
    const int64_t lo = min(ntasks, (int64_t)tid * per), hi = min(ntasks, lo + per);
    unsigned long long s = 0;
    for (int64_t t = lo; t < hi; ++t) s += sb.task_cnt[t] - sb.task_prev[t];
    part[tid] = s;
    __syncthreads();
    block_inclusive_scan(part);
    unsigned long long run = part[tid] - s;
    for (int64_t t = lo; t < hi; ++t) {
        const unsigned long long c = sb.task_cnt[t];
        sb.seg_off[t] = next_base + (int64_t)run;
        sb.seg_cur[t] = 0ull;
        run += c - sb.task_prev[t];
        sb.task_prev[t] = c;
    }
}

// one workgroup, for a level that is not regrouped: task_prev = task_cnt, so
// the next regrouping sees only the growth of its own level (same task
// partition over the threads as greedy_segments, so no barrier is needed
// between the two)
static __device__ void greedy_mark_prev(const SearchBufs &sb, int64_t ntasks) {
    const int64_t per = (ntasks + blockDim.x - 1) / blockDim.x;
    const int64_t lo = min(ntasks, (int64_t)threadIdx.x * per), hi = min(ntasks, lo + per);
    for (int64_t t = lo; t < hi; ++t) sb.task_prev[t] = sb.task_cnt[t];
}

// regroup the unsorted level [lo, hi) by task into the item arrays; one
// cursor atomic per run of equal tasks
template <typename O>
__device__ void greedy_regroup(const SearchBufs &sb, int64_t lo, int64_t hi) {
    const int lane = lane_id();
    const int64_t gw = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int64_t tw = (int64_t)gridDim.x * (blockDim.x >> 6);
    const O *ud = (const O *)sb.u_dist;
    O *idist = (O *)sb.item_dist;
    for (int64_t c = lo + gw * 64; c < hi; c += tw * 64) {
        const int64_t i = c + lane;
        const bool valid = i < hi;
        const unsigned long long key = valid ? sb.u_key[i] : ~0ull;
        const int32_t t = valid ? (int32_t)(key >> 32) : -1;
        const int32_t tprev = __shfl_up(t, 1);
        const bool head = valid && (lane == 0 || tprev != t);
        const unsigned long long hm = __ballot(head);
        const unsigned long long vm = __ballot(valid);
        unsigned long long o = 0;
        int hl = 0;
        if (valid) {
            hl = 63 - __clzll((long long)(hm & ((2ull << lane) - 1ull)));
        }
        if (head) {
            const unsigned long long later = hm & ~((2ull << lane) - 1ull);
            const int end = later ? __ffsll((long long)later) - 1 : 64 - __clzll((long long)vm);
            o = atomicAdd(&sb.seg_cur[t], (unsigned long long)(end - lane));
        }
        const unsigned long long ob = __shfl(o, hl);
        const int64_t pos = valid ? sb.seg_off[t] + (int64_t)ob + (lane - hl) : -1;
        if (valid && pos >= lo && pos < hi) {
            sb.item_key[pos] = key;
            idist[pos] = ud[i];
        }
    }
}

// Grid-wide barrier of a cooperative launch (every workgroup resident),
// crossed for the k-th time (k >= 1).  Workgroup g arrives on group counter
// g % BARRIER_GROUPS; the last arrival of a group (its returning add reaches
// k times the group's size) arrives on the top counter, and every workgroup
// waits for the top counter to reach k times the number of groups.  Counters
// only grow, so the k-th crossing's targets are exact.  Arrivals on one
// counter are serialized, so the groups cut the serial part from gridDim.x
// atomics to gridDim.x / BARRIER_GROUPS plus BARRIER_GROUPS.  The agent-scope
// release before arriving and acquire after leaving make the workgroup's
// writes visible to every other workgroup, as a grid sync must; the last
// arrival of a group also acquires what its group released before it passes
// it on.  The spin is bounded: past the limit the search is marked as failed
// (overflow bit 256) instead of waiting forever.
__device__ __forceinline__ void grid_barrier(unsigned long long *groups, unsigned long long *top,
                                             unsigned long long k, unsigned long long *overflow) {
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned ng = gridDim.x < BARRIER_GROUPS ? gridDim.x : BARRIER_GROUPS;
        const unsigned g = blockIdx.x % ng;
        const unsigned long long gsize = gridDim.x / ng + (g < gridDim.x % ng ? 1u : 0u);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const unsigned long long old =
            __hip_atomic_fetch_add(groups + (size_t)g * CTR_STRIDE, 1ull, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        if (old + 1 == k * gsize) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "agent");
            __hip_atomic_fetch_add(top, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const unsigned long long target = k * ng;
        long spins = 0;
        while (__hip_atomic_load(top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > (1l << 26)) {
                atomicOr(overflow, OVERFLOW_BARRIER);
                break;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
}

template <int DTYPE, int CPL, int G>
__global__ __launch_bounds__((greedy_waves<DTYPE, CPL>() * 64)) void k_greedy(GreedyArgs a) {
    using D = typename DistOf<DTYPE>::T;
    using O = typename DistOf<DTYPE>::O;
    constexpr int GREEDY_WAVES = greedy_waves<DTYPE, CPL>();
    extern __shared__ __align__(16) uint8_t greedy_smem[];
    GreedyLds<D, O, GREEDY_WAVES> &L = *reinterpret_cast<GreedyLds<D, O, GREEDY_WAVES> *>(greedy_smem);
    unsigned long long barriers = 0;
    auto grid_sync = [&]() {
        ++barriers;
        grid_barrier(&a.sb.counters[CTR_BARRIER_GROUP], &a.sb.counters[CTR_BARRIER], barriers,
                     &a.sb.counters[CTR_OVERFLOW]);
    };
    const int lane = lane_id();
    const int wid = threadIdx.x >> 6;
    const DevIndex &ix = a.ix;
    const int R = ix.R;
    uint32_t *qi = L.ci[wid]; // candidate queue: ids inserted into the global set
    const int64_t hmask = a.sb.hash_cap - 1;
    const int64_t ntasks = (int64_t)a.sb.counters[CTR_TASKS];
    uint32_t set_ops = 0; // global set updates of the wave (a wave-uniform count)
    // phase timestamps (block 0, one lane): kernel start, then per level the
    // ends of expansion, segment scan and regroup
    const bool clock_lane = blockIdx.x == 0 && threadIdx.x == 0;
    auto stamp = [&](int lv, int k) {
        if (clock_lane && lv < LEVEL_CLOCKS) a.sb.level_clock[1 + 3 * lv + k] = wall_clock64();
    };
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < 1 + 3 * LEVEL_CLOCKS; i += blockDim.x)
            a.sb.level_clock[i] = i == 0 ? wall_clock64() : 0ull;
    int64_t base = 0;
    int lvl = 0;
    bool grouped = true;
    const int64_t regroup_min = 512 * (int64_t)gridDim.x;
    // Level 0: the seeds (N of each expanding task), written by the beam
    // kernel.  Level 1: what the task-local kernel found and expanded.  Level
    // 2: the unexpanded points it handed on, and what the seeds of the tasks
    // it left find here.
    auto level_size = [&](int l) {
        return (int64_t)__hip_atomic_load(&a.sb.level_cnt[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const bool local = a.sb.local_grid > 0;
    const int64_t left = local ? (int64_t)a.sb.counters[CTR_LEFT] : ntasks;
    const int64_t spilled = local ? (int64_t)a.sb.counters[CTR_SPILL] : 0;
    const int64_t size0 = level_size(0), size1 = local ? level_size(1) : 0;
    if (local && left == 0 && spilled == 0) {
        if (clock_lane) {
            a.sb.counters[CTR_LEVELS] = size0 > 0 ? 2 : 0;
            a.sb.counters[CTR_GREEDY_ITEMS] = (unsigned long long)(size0 + size1);
        }
        return;
    }
    {
        // the seeds join the (task, id) set before any expansion (the bitmaps
        // were cleared by an earlier kernel: its end orders those stores
        // before these updates); points handed on move to level 2
        const int64_t c0 = min(size0, a.sb.item_cap), b2 = size0 + size1;
        bool full = false;
        const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
        if (left > 0)
            for (int64_t i = i0; i < c0; i += stride) {
                const unsigned long long key = a.sb.item_key[i];
                const int32_t t = (int32_t)(key >> 32);
                if (t < 0 || t >= ntasks || a.sb.task_expand[t] != 1) continue;
                bool f = false;
                tset_add(a.sb, hmask, t, (uint32_t)key, f);
                if (f) {
                    a.sb.task_trunc[t] = 1;
                    full = true;
                }
            }
        for (int64_t i = i0; i < spilled; i += stride)
            if (b2 + i < a.sb.item_cap) {
                a.sb.u_key[b2 + i] = a.sb.item_key[a.sb.item_cap - 1 - i];
                ((O *)a.sb.u_dist)[b2 + i] = ((const O *)a.sb.item_dist)[a.sb.item_cap - 1 - i];
            }
        if (clock_lane && spilled > 0) atomicAdd(&a.sb.level_cnt[2], (unsigned long long)spilled);
        if (__ballot(full) && lane == 0) atomicOr(&a.sb.counters[CTR_OVERFLOW], 8ull);
        grid_sync();
    }
    for (; lvl < a.sb.max_levels - 1;) {
        const int64_t cnt = lvl == 0 ? size0 + size1 : level_size(lvl);
        if (cnt == 0) break;
        const int nx = lvl == 0 && local ? 2 : lvl + 1;
        const int64_t next_base = base + cnt;
        for (int i = threadIdx.x; i < GREEDY_CACHE; i += blockDim.x) L.cache[i] = ~0ull;
        if (lane == 0) L.st_n[wid] = 0;
        __syncthreads();
        // where this level's items are: the item arrays (level 0, or regrouped)
        // or the unsorted level as emitted
        const unsigned long long *src_key = grouped ? a.sb.item_key : a.sb.u_key;
        // this workgroup's block of the level (items beyond item_cap were dropped)
        // (level 0: the seeds, without level 1)
        const int64_t avail = lvl == 0 ? (left > 0 ? min(size0, a.sb.item_cap) : 0)
                                       : max((int64_t)0, min(cnt, a.sb.item_cap - base));
        const int64_t per = (avail + gridDim.x - 1) / gridDim.x;
        const int64_t i0 = min(avail, xcd_block() * per), i1 = min(avail, i0 + per);

        // the queue holds candidates of one task, `qtask`, whose query is in qr
        int qn = 0;
        int32_t qtask = -1;
        unsigned long long run_evals = 0, run_rechk = 0;
        QThresh th{};
        QueryRegs<DTYPE, CPL, G> qr;

        // distances of the queued candidates in one gather; in-range ones are
        // staged for the next level
        auto flush = [&]() __attribute__((always_inline)) {
            const int k = qn;
            if (k == 0) return;
            for (int b0 = 0; b0 < k; b0 += 64) {
                const int kb = min(64, k - b0);
                bool inr = false;
                O myd = dmax<O>();
                uint32_t myi = 0;
                decide64<DTYPE, CPL, G>(ix, qr, th, qi + b0, kb, L.xi[wid], myd, myi, inr, run_rechk);
                const unsigned long long im = __ballot(inr);
                const int m = __popcll(im);
                if (m == 0) continue;
                int sn = L.st_n[wid];
                if (sn + m > GREEDY_STAGE) {
                    // stage full: reserve for it now
                    unsigned long long o = 0;
                    if (lane == 0) o = atomicAdd(&a.sb.level_cnt[nx], (unsigned long long)sn);
                    o = __shfl(o, 0);
                    greedy_emit(L, wid, sn, next_base + (int64_t)o, a.sb);
                    wave_sync();
                    sn = 0;
                }
                if (inr) {
                    const int o = sn + mbcnt(im);
                    L.st_id[wid][o] = myi;
                    L.st_task[wid][o] = qtask;
                    L.st_d[wid][o] = myd;
                }
                wave_sync();
                if (lane == 0) L.st_n[wid] = sn + m;
                wave_sync();
            }
            qn = 0;
        };
        auto close_task = [&]() __attribute__((always_inline)) {
            if (qtask >= 0 && lane == 0) {
                if (run_evals) atomicAdd(&a.sb.task_evals[qtask], run_evals);
                if (run_rechk) atomicAdd(&a.sb.task_rechk[qtask], run_rechk);
            }
            run_evals = 0;
            run_rechk = 0;
        };
        // queue the lanes' ids in `mask` (new members of task t's set)
        auto enqueue = [&](int32_t t, unsigned long long mask, bool mine, int32_t f) __attribute__((always_inline)) {
            if (t != qtask) {
                flush();
                close_task();
                qtask = t;
                const int32_t q = a.sb.task_q[t];
                th = a.sb.qth[q];
                qr.load(a.sb.qpad + (size_t)q * qrow_stride<DTYPE>(ix), ix);
            }
            if (mine) qi[qn + mbcnt(mask)] = (uint32_t)f;
            wave_sync();
            const int k = __popcll(mask);
            qn += k;
            run_evals += (unsigned long long)k;
        };

        // Item j of this wave is i0 + wid + GREEDY_WAVES * j; items are taken
        // in pairs, in a four-stage software pipeline: item records three pairs
        // ahead, adjacency rows two pairs ahead, the set updates one pair
        // ahead of the pair whose results are consumed.  Loads are issued
        // without branches and their values are first used one stage later,
        // so a wave keeps several round trips to memory in flight.
        const int64_t nidx = ix.n;
        auto load_item = [&](int64_t it, int32_t &t, int32_t &p, bool &in) {
            in = it < i1;
            const int64_t k = in ? base + it : 0;
            const unsigned long long key = src_key[k];
            t = (int32_t)(key >> 32);
            p = (int32_t)(uint32_t)key;
        };
        // sanitises the item (items beyond item_cap are never written) and
        // loads its expansion flag and adjacency row
        auto load_adj = [&](bool in, int32_t t, int32_t p, int32_t &tv, int32_t &f, int &e) {
            const bool v = in && t >= 0 && t < ntasks && p >= 0 && (int64_t)p < nidx;
            tv = v ? t : -1;
            const int32_t ts = v ? t : 0, ps = v ? p : 0;
            e = a.sb.task_expand[ts];
            if (lvl == 0) e = e == 1; // 2: the seeds were expanded by the task-local kernel
            f = ix.adj[(size_t)ps * (size_t)R + (size_t)max(0, min(lane, R - 1))];
        };
        // the set update of a pair: neighbours not yet known to the workgroup
        // cache go to the global set (bitmap words are returned for the
        // consume stage; hash-table tasks are decided here)
        struct Pend {
            uint32_t oA, oB;
            bool bA, bB, xA, xB;
        };
        auto issue = [&](int32_t tA, int32_t fA, int eA, int32_t tB, int32_t fB, int eB, Pend &P) __attribute__((always_inline)) {
            const bool okA = tA >= 0 && eA && lane < R && fA >= 0;
            const bool okB = tB >= 0 && eB && lane < R && fB >= 0;
            const unsigned long long keyA = ((unsigned long long)(uint32_t)tA << 32) | (uint32_t)fA;
            const unsigned long long keyB = ((unsigned long long)(uint32_t)tB << 32) | (uint32_t)fB;
            const bool cA = okA && !wg_cache_seen(L.cache, keyA);
            const bool cB = okB && !wg_cache_seen(L.cache, keyB);
            P.bA = cA && tA < a.sb.bm_tasks;
            P.bB = cB && tB < a.sb.bm_tasks;
            set_ops += (uint32_t)(__popcll(__ballot(cA)) + __popcll(__ballot(cB)));
            P.oA = ~0u;
            P.oB = ~0u;
            if (P.bA) P.oA = atomicOr(&a.sb.bm[(int64_t)tA * a.sb.bm_words + ((uint32_t)fA >> 5)],
                                      1u << (fA & 31));
            if (P.bB) P.oB = atomicOr(&a.sb.bm[(int64_t)tB * a.sb.bm_words + ((uint32_t)fB >> 5)],
                                      1u << (fB & 31));
            const bool hA = cA && !P.bA, hB = cB && !P.bB;
            P.xA = false;
            P.xB = false;
            bool full = false;
            if (__ballot(hA || hB)) {
                gset_insert2(a.sb.hash, hmask, keyA, hA, keyB, hB, P.xA, P.xB, full);
                if (full) {
                    if (hA) a.sb.task_trunc[tA] = 1;
                    if (hB) a.sb.task_trunc[tB] = 1;
                }
                if (__ballot(full) && lane == 0) atomicOr(&a.sb.counters[CTR_OVERFLOW], 8ull);
            }
        };
        auto consume = [&](int32_t tA, int32_t fA, int32_t tB, int32_t fB, const Pend &P) __attribute__((always_inline)) {
            const bool nA = P.bA ? !(P.oA & (1u << (fA & 31))) : P.xA;
            const bool nB = P.bB ? !(P.oB & (1u << (fB & 31))) : P.xB;
            const unsigned long long mA = __ballot(nA), mB = __ballot(nB);
            if (mA) enqueue(tA, mA, nA, fA);
            if (mB) enqueue(tB, mB, nB, fB);
            if (qn >= 64) flush();
        };
        const int64_t S = GREEDY_WAVES;
        int64_t it = i0 + wid;
        // stage 3 (consume), 2 (issue), 1 (adjacency), 0 (items)
        int32_t tA3, fA3, tB3, fB3;
        int32_t tA2, fA2, tB2, fB2;
        int eA2, eB2;
        int32_t tA1, pA1, tB1, pB1, tA0, pA0, tB0, pB0;
        bool iA1, iB1, iA0, iB0;
        Pend P3;
        {
            int32_t t, p;
            bool in;
            int e;
            load_item(it, t, p, in);
            load_adj(in, t, p, tA3, fA3, e);
            int32_t tb, pb;
            bool inb;
            int eb;
            load_item(it + S, tb, pb, inb);
            load_adj(inb, tb, pb, tB3, fB3, eb);
            issue(tA3, fA3, e, tB3, fB3, eb, P3);
        }
        {
            int32_t t, p, tb, pb;
            bool in, inb;
            load_item(it + 2 * S, t, p, in);
            load_item(it + 3 * S, tb, pb, inb);
            load_adj(in, t, p, tA2, fA2, eA2);
            load_adj(inb, tb, pb, tB2, fB2, eB2);
        }
        load_item(it + 4 * S, tA1, pA1, iA1);
        load_item(it + 5 * S, tB1, pB1, iB1);
        for (; it < i1; it += 2 * S) {
            load_item(it + 6 * S, tA0, pA0, iA0);
            load_item(it + 7 * S, tB0, pB0, iB0);
            int32_t tAn, fAn, tBn, fBn;
            int eAn, eBn;
            load_adj(iA1, tA1, pA1, tAn, fAn, eAn);
            load_adj(iB1, tB1, pB1, tBn, fBn, eBn);
            Pend P2;
            issue(tA2, fA2, eA2, tB2, fB2, eB2, P2);
            consume(tA3, fA3, tB3, fB3, P3);

            tA3 = tA2; fA3 = fA2; tB3 = tB2; fB3 = fB2; P3 = P2;
            tA2 = tAn; fA2 = fAn; eA2 = eAn; tB2 = tBn; fB2 = fBn; eB2 = eBn;
            tA1 = tA0; pA1 = pA0; iA1 = iA0; tB1 = tB0; pB1 = pB0; iB1 = iB0;
        }
        flush();
        close_task();
        // one reservation per workgroup for what the waves still hold
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long tot = 0;
            for (int w = 0; w < GREEDY_WAVES; ++w) tot += (unsigned long long)L.st_n[w];
            L.wg_base = tot ? atomicAdd(&a.sb.level_cnt[nx], tot) : 0ull;
        }
        __syncthreads();
        {
            int64_t off = (int64_t)L.wg_base;
            for (int w = 0; w < wid; ++w) off += L.st_n[w];
            const int sn = L.st_n[wid];
            if (sn > 0) greedy_emit(L, wid, sn, next_base + off, a.sb);
        }
        grid_sync();
        stamp(lvl, 0);
        // regroup the next level by task
        const int64_t ncnt = level_size(nx);
        if (ncnt == 0) {
            lvl = nx;
            break;
        }
        // levels below 512 items per workgroup are expanded as emitted (their
        // items are moved to the item arrays at the end): regrouping them costs
        // two grid barriers and a pass, more than their locality gains back
        grouped = ncnt >= regroup_min;
        if (!grouped && blockIdx.x == 0) greedy_mark_prev(a.sb, ntasks);
        if (grouped) {
            if (blockIdx.x == 0) greedy_segments(L.part, a.sb, ntasks, next_base);
            grid_sync();
            stamp(lvl, 1);
            const int64_t stored = max((int64_t)0, min(ncnt, a.sb.item_cap - next_base));
            greedy_regroup<O>(a.sb, next_base, next_base + stored);
            grid_sync();
            stamp(lvl, 2);
        }
        base = next_base;
        lvl = nx;
    }
    // the set-operation count: one global atomic per workgroup (one per wave,
    // all arriving together at the end, would serialize on the counter)
    __syncthreads();
    if (threadIdx.x == 0) L.wg_base = 0ull;
    __syncthreads();
    if (lane == 0 && set_ops) atomicAdd(&L.wg_base, (unsigned long long)set_ops);
    __syncthreads();
    if (threadIdx.x == 0 && L.wg_base) atomicAdd(&a.sb.counters[CTR_SET_OPS], L.wg_base);
    // move the levels that were expanded as emitted into the item arrays (the
    // kernel's end orders these writes before the finalisation)
    {
        int64_t b0 = 0;
        const O *ud = (const O *)a.sb.u_dist;
        O *idist = (O *)a.sb.item_dist;
        // (level lvl is empty, except when the level limit stopped the loop:
        // then its points were never expanded and their tasks are truncated)
        const bool limit = lvl == a.sb.max_levels - 1;
        for (int l = 0; l <= lvl && l < a.sb.max_levels; ++l) {
            const int64_t c = (int64_t)__hip_atomic_load(&a.sb.level_cnt[l], __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
            const int64_t lo = b0, hi = min(b0 + c, a.sb.item_cap);
            b0 += c;
            const bool in_items = l == 0 || (local && l == 1) || c >= regroup_min;
            if (limit && l == lvl)
                for (int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi;
                     i += (int64_t)gridDim.x * blockDim.x)
                    a.sb.task_trunc[(int32_t)((in_items ? a.sb.item_key[i] : a.sb.u_key[i]) >> 32)] = 1;
            if (in_items) continue;
            for (int64_t i = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < hi;
                 i += (int64_t)gridDim.x * blockDim.x) {
                a.sb.item_key[i] = a.sb.u_key[i];
                idist[i] = ud[i];
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.sb.counters[CTR_LEVELS] = (unsigned long long)lvl;
        unsigned long long items = 0;
        for (int l = 0; l <= lvl && l < a.sb.max_levels; ++l)
            items += __hip_atomic_load(&a.sb.level_cnt[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a.sb.counters[CTR_GREEDY_ITEMS] = items;
        if (lvl == a.sb.max_levels - 1 &&
            __hip_atomic_load(&a.sb.level_cnt[lvl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
            atomicOr(&a.sb.counters[CTR_OVERFLOW], 16ull);
    }
}

// --------------------------------------------------------------------------
// greedy phase, first part: one workgroup per task
// --------------------------------------------------------------------------

// Algorithm 2 of one task inside one workgroup.  The set of evaluated points
// is a bitmap of n bits in LDS (up to 1.1M points: 160 KB a CU), so a probe is
// one LDS atomic; there are no levels, no grid barrier, no bitmap in memory
// to clear.  Waves take the found points in the order of their list: wave
// tickets run through the seeds, then through the list, and a wave whose
// ticket is ahead of the list waits until the point is there or every point
// taken has been finished.
//
// A large ball would keep one workgroup busy while the rest of the GPU is idle,
// so a task is handed on when few workgroups are busy (local_busy) and its
// backlog is long, or when its list is full: the bitmap goes to memory (or its
// ids to the hash table) and the unexpanded points to the level kernel, which
// spreads them over the GPU.
//
// What bounds it: a wave's chain of two reads (adjacency row, base rows) per
// point, with 8 to 16 waves a CU.  The level kernel alone spends most of its
// time on atomics of the memory's set (13 to 16 G/s reached) and, on small
// levels, on barriers.  Both kernels, before and now: 10,000 queries of the 1M
// x 128 uint8 Vamana workload (642K points, lists up to 6.8K) 0.71 -> 0.53 ms;
// 156K points, lists up to 1.4K 0.67 -> 0.26 ms; 1M x 96 bfloat16 pass, 3.6M
// points 13.1 -> 6.0 ms; 100K x 768 8-bit pass, 45K points 1.16 -> 0.56 ms.
// Handing on at a backlog of 384 or 1,024 points took 1 and 4% longer on the
// first, with half or three quarters of the workgroups still busy 5 and 9%.
constexpr int LOCAL_BACKLOG = 192;   // points waiting, from which the level kernel is worth its start
constexpr int LOCAL_WAIT = 512;      // the same while more workgroups are busy (integer data)

// Whether the task-local kernel runs, with how many workgroups and how long a
// list each (a list's distances lie in the finalization's item_cap entries,
// which are free until then).  It needs the bitmap and the list in LDS, a
// list some way above the margin, and a workgroup for every CU or query.
inline void plan_local(SearchBufs &sb, int64_t n, int64_t nq, int num_cus) {
    sb.local_grid = sb.local_cap = 0;
    const int64_t words = bitmap_words(n), least = LOCAL_LEAST;
    const int64_t lds = 160 * 1024, fix = words * 4 + LOCAL_WAVES * 64 * 8 + 512;
    if (nq <= 0 || fix + least * 4 > lds) return;
    const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(4, lds / (fix + LOCAL_LIST * 4)));
    const int64_t grid = std::min(std::min(nq, per_cu * num_cus), sb.item_cap / least);
    if (grid < std::min<int64_t>(nq, num_cus)) return;
    const int64_t list = std::min<int64_t>(LOCAL_LIST, (lds / per_cu - fix) / 4);
    sb.bm_words = words;
    sb.local_grid = (int32_t)grid;
    sb.local_full = grid == per_cu * num_cus;
    sb.local_cap = (int32_t)(std::min<int64_t>(list, sb.item_cap / grid) & ~3ll);
}

// Workgroups still busy at which tasks are handed on, from a backlog of
// LOCAL_BACKLOG and of LOCAL_WAIT points.  With a workgroup for all that the GPU
// holds: a quarter of them.  With fewer tasks than that the level kernel's own
// time, 100 us and more, has to be gained on them alone: a workgroup expands 2
// to 6 points a us on float data, where it pays for up to a quarter of the CUs,
// and 8 on integer data, where it does for a few.  Calls of 12 queries with
// 1,500 and 4,000 results each, level kernel alone / handed on when three
// quarters of these 12 are done / now: 1M x 128 uint8 544 / 381 / 498 and 738 /
// 661 / 657 us, 200K x 96 bfloat16 pass 537 / 578 / 438 and 675 / 1,253 / 534,
// 100K x 768 8-bit pass 1,094 / 1,241 / 554 and 1,547 / 2,405 / 680.
inline LocalBusy local_busy(bool full, int grid, int num_cus, bool integer) {
    if (full) return {grid / 4, grid / 4};
    return integer ? LocalBusy{num_cus / 64, num_cus / 16} : LocalBusy{num_cus / 4, num_cus / 4};
}

struct LocalTask {
    int head, tail, done, stop; // tickets given, points found, points finished
    int task, ns, seeds, cs, cd; // seeds: of the points finished
    unsigned evals, rechk;
    unsigned long long base_d, base_s;
    long long keep_d, keep_s;
};
inline size_t local_lds(int64_t bm_words, int cap, int gw, bool approx) {
    return (size_t)bm_words * 4 + (size_t)cap * 4 + (size_t)gw * 64 * (approx ? 8 : 4) + sizeof(LocalTask);
}

// waves per workgroup: as many as the registers of the distance code leave
template <int DTYPE, int CPL> constexpr int local_waves() {
    return dfloat(DTYPE) ? (dbase(DTYPE) == RR_SQ8X && CPL >= 3 ? 8 : 12) : CPL >= 6 ? 12 : 16;
}

template <int DTYPE, int CPL, int G>
__global__ __launch_bounds__((local_waves<DTYPE, CPL>() * 64)) void k_greedy_local(GreedyArgs a) {
    using O = typename DistOf<DTYPE>::O;
    constexpr int GW = local_waves<DTYPE, CPL>();
    extern __shared__ __align__(16) uint8_t local_smem[];
    uint32_t *const bm = reinterpret_cast<uint32_t *>(local_smem);
    const int64_t words = a.sb.bm_words;
    const int cap = a.sb.local_cap;
    volatile uint32_t *const ids = bm + words;
    const int lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t *const ci = bm + words + cap + wid * 64;
    uint32_t *const xi = bm + words + cap + (GW + wid) * 64; // approximate passes
    LocalTask &T = *reinterpret_cast<LocalTask *>(bm + words + cap + (dapprox(DTYPE) ? 2 : 1) * GW * 64);
    volatile int *const v_tail = &T.tail, *const v_done = &T.done, *const v_seeds = &T.seeds, *const v_stop = &T.stop;
    const DevIndex &ix = a.ix;
    const int R = ix.R;
    const int64_t ntasks = (int64_t)a.sb.counters[CTR_TASKS];
    const int64_t size0 = min((int64_t)a.sb.level_cnt[0], a.sb.item_cap);
    O *const idist = (O *)a.sb.item_dist;
    O *const sc = (O *)a.sb.seg_dists + (int64_t)blockIdx.x * cap; // the list's distances
    unsigned long long *const queue = &a.sb.counters[CTR_LOCAL_QUEUE];
    // tickets given out when few enough workgroups are busy
    const int64_t idle = ntasks + (int64_t)gridDim.x - a.busy.low, idle_long = ntasks + (int64_t)gridDim.x - a.busy.high;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.sb.level_clock[LOCAL_CLOCK] = wall_clock64();

    for (;;) {
        if (threadIdx.x == 0) {
            T.task = (int)atomicAdd(queue, 1ull);
            T.head = T.tail = T.done = T.stop = 0;
            T.evals = T.rechk = 0u;
            T.ns = T.seeds = T.cs = T.cd = 0;
        }
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(T.task);
        if (t >= ntasks) break;
        const int nseed = (int)a.sb.task_cnt[t];
        if (!a.sb.task_expand[t] || nseed > LOCAL_SEEDS) {
            if (a.sb.task_expand[t]) {
                // left to the level kernel, which starts from an empty set
                if (t < a.sb.bm_tasks)
                    for (int64_t i = threadIdx.x; i < words / 4; i += blockDim.x)
                        reinterpret_cast<uint4 *>(a.sb.bm + t * words)[i] = make_uint4(0u, 0u, 0u, 0u);
                if (threadIdx.x == 0) atomicAdd(&a.sb.counters[CTR_LEFT], 1ull);
            }
            __syncthreads(); // T is written again
            continue;
        }
        const int64_t seed0 = a.sb.task_out[t];
        const int32_t q = __builtin_amdgcn_readfirstlane(a.sb.task_q[t]);
        for (int64_t i = threadIdx.x; i < words / 4; i += blockDim.x)
            reinterpret_cast<uint4 *>(bm)[i] = make_uint4(0u, 0u, 0u, 0u);
        for (int i = threadIdx.x; i < cap; i += blockDim.x) ids[i] = RR_EMPTY32;
        const QThresh th = a.sb.qth[q];
        QueryRegs<DTYPE, CPL, G> qr;
        qr.load(a.sb.qpad + (size_t)q * qrow_stride<DTYPE>(ix), ix);
        __syncthreads();
        if (threadIdx.x < nseed) {
            const uint32_t id = (uint32_t)a.sb.item_key[seed0 + threadIdx.x];
            atomicOr(&bm[id >> 5], 1u << (id & 31));
        }
        __syncthreads();
        unsigned evals = 0;
        unsigned long long rechk = 0;
        // a wave takes its next ticket, and loads its adjacency row if the
        // point is there already, before it evaluates the current neighbours
        auto ticket = [&]() {
            int i = 0;
            if (lane == 0) i = atomicAdd(&T.head, 1);
            return (int)__builtin_amdgcn_readfirstlane(i);
        };
        auto row = [&](uint32_t p) { return ix.adj[(uint64_t)p * (uint32_t)R + max(0, min(lane, R - 1))]; };
        int i = ticket();
        uint32_t np = RR_EMPTY32; // the ticket's point, if it is known
        int32_t nf = -1;          // and its row
        for (;;) {
            uint32_t p = np;
            const int k0 = i - nseed;
            if (k0 < 0) {
                if (p == RR_EMPTY32) p = (uint32_t)a.sb.item_key[seed0 + i];
            } else {
                uint32_t v = RR_EMPTY32;
                for (;;) {
                    if (*v_stop) break;
                    if (k0 < cap) v = ids[k0];
                    if (v != RR_EMPTY32) break;
                    // every point found is finished: no more will come (`done`
                    // is read before `tail`, and a wave adds to `tail` before
                    // it adds to `done`)
                    const int d = *v_done;
                    if (d == nseed + *v_tail) break;
                    __builtin_amdgcn_s_sleep(1);
                }
                p = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
                if (p == RR_EMPTY32) break;
                // now and then: how many workgroups are busy?  (the others have
                // taken one ticket past the end each)
                if ((k0 & 31) == 0 && *v_tail - k0 > LOCAL_BACKLOG) {
                    const int64_t given = (int64_t)__hip_atomic_load(queue, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (given >= (*v_tail - k0 > LOCAL_WAIT ? idle_long : idle) && lane == 0) *v_stop = 1;
                }
            }
            const int32_t f = np == p ? nf : row(p);
            bool cand = false;
            if (lane < R && f >= 0) {
                const uint32_t bit = 1u << (f & 31);
                cand = !(atomicOr(&bm[(uint32_t)f >> 5], bit) & bit);
            }
            const unsigned long long cm = __ballot(cand);
            const int k = __popcll(cm);
            evals += (unsigned)k;
            const int ni = ticket();
            np = RR_EMPTY32;
            if (ni < nseed) np = (uint32_t)a.sb.item_key[seed0 + ni];
            else if (ni - nseed < cap) np = (uint32_t)__builtin_amdgcn_readfirstlane((int)ids[ni - nseed]);
            if (np != RR_EMPTY32) nf = row(np);
            if (k > 0) {
                if (cand) ci[mbcnt(cm)] = (uint32_t)f;
                wave_sync();
                bool in = false;
                O d = dmax<O>();
                uint32_t id = 0;
                decide64<DTYPE, CPL, G>(ix, qr, th, ci, k, xi, d, id, in, rechk);
                wave_sync();
                const unsigned long long im = __ballot(in);
                if (im) {
                    const int m = __popcll(im);
                    // (read before the points are added: local_margin)
                    const int open = nseed - __builtin_amdgcn_readfirstlane(*v_seeds);
                    wave_sync();
                    int pos = 0;
                    if (lane == 0) pos = atomicAdd(&T.tail, m);
                    pos = __builtin_amdgcn_readfirstlane(pos);
                    if (pos + m > cap - local_margin(GW, open) && lane == 0) *v_stop = 1;
                    const int o = pos + mbcnt(im);
                    if (in) {
                        sc[o] = d;
                        ids[o] = id; // (o < cap: local_margin)
                    }
                }
            }
            wave_sync();
            if (lane == 0) {
                if (i >= nseed) ids[i - nseed] = p | 0x80000000u; // expanded
                else atomicAdd(&T.seeds, 1);
                atomicAdd(&T.done, 1);
            }
            i = ni;
        }
        if (lane == 0) {
            atomicAdd(&T.evals, evals);
            if (rechk) atomicAdd(&T.rechk, (unsigned)rechk);
        }
        __syncthreads();
        // the list: expanded points become items of level 1, the others are
        // handed on from the top of the item arrays
        const int n = T.tail;
        const bool stopped = T.stop != 0;
        if (stopped) {
            int u = 0;
            for (int i = threadIdx.x; i < n; i += blockDim.x) u += ids[i] & 0x80000000u ? 0 : 1;
            if (u) atomicAdd(&T.ns, u);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            const long long ns = T.ns, nd = n - ns;
            // both parts fit between the seeds and the end of the arrays, or
            // the rest is dropped
            const long long old = n ? (long long)atomicAdd(&a.sb.counters[CTR_LOCAL_ITEMS], (unsigned long long)n) : 0;
            const long long room = max(0ll, (long long)(a.sb.item_cap - size0) - old);
            T.keep_d = min(nd, room);
            T.keep_s = min(ns, room - T.keep_d);
            T.base_d = T.keep_d ? atomicAdd(&a.sb.level_cnt[1], (unsigned long long)T.keep_d) : 0ull;
            T.base_s = T.keep_s ? atomicAdd(&a.sb.counters[CTR_SPILL], (unsigned long long)T.keep_s) : 0ull;
            if (T.keep_d + T.keep_s < n) {
                a.sb.task_trunc[t] = 1;
                atomicOr(&a.sb.counters[CTR_OVERFLOW], 4ull);
            }
            a.sb.task_cnt[t] = (unsigned long long)(nseed + T.keep_d + T.keep_s);
            a.sb.task_prev[t] = (unsigned long long)(nseed + T.keep_d);
            a.sb.task_evals[t] = T.evals;
            a.sb.task_rechk[t] = T.rechk;
            a.sb.task_expand[t] = 2;
        }
        __syncthreads();
        const unsigned long long tk = (unsigned long long)(uint32_t)t << 32;
        for (int i = threadIdx.x; i < n; i += blockDim.x) {
            const uint32_t v = ids[i];
            const bool on = stopped && !(v & 0x80000000u);
            const int j = !stopped ? i : atomicAdd(on ? &T.cs : &T.cd, 1);
            if (j >= (on ? T.keep_s : T.keep_d)) continue;
            const int64_t o = on ? a.sb.item_cap - 1 - (int64_t)T.base_s - j : size0 + (int64_t)T.base_d + j;
            a.sb.item_key[o] = tk | (v & 0x7fffffffu);
            idist[o] = sc[i];
        }
        if (T.keep_s > 0) {
            if (t < a.sb.bm_tasks) {
                for (int64_t i = threadIdx.x; i < words / 4; i += blockDim.x)
                    reinterpret_cast<uint4 *>(a.sb.bm + t * words)[i] = reinterpret_cast<const uint4 *>(bm)[i];
            } else {
                bool full = false;
                for (int64_t i = threadIdx.x; i < words; i += blockDim.x)
                    for (uint32_t w = bm[i]; w; w &= w - 1)
                        gset_insert(a.sb.hash, a.sb.hash_cap - 1, tk | (uint32_t)(32 * i + __ffs((int)w) - 1), full);
                if (full) {
                    a.sb.task_trunc[t] = 1;
                    atomicOr(&a.sb.counters[CTR_OVERFLOW], 8ull);
                }
            }
        }
        __syncthreads(); // T and the list are written again
    }
}

// ---- finalisation of the greedy phase: group items per task, sort, emit ----
struct SlotArgs {
    const int32_t *qlist = nullptr;
    int64_t nwork = 0;
    BeamState *state = nullptr;
    void *st_d = nullptr;
    uint32_t *st_i = nullptr;
    int32_t step_budget = 0;
    int32_t probe_step = 0;
    double *probe_m = nullptr;
    int8_t *probe_f = nullptr;
};

template <int DTYPE, int CPL, int G>
static hipError_t run_beam(const DevIndex &ix, int64_t nq, const SearchCfg &cfg, SearchBufs &sb,
                           int num_cus, hipStream_t s, const SlotArgs &sl) {
    using D = typename DistOf<DTYPE>::T;
    BeamArgs a;
    a.ix = ix;
    a.nq = nq;
    a.cfg = cfg;
    a.sb = sb;
    a.qlist = sl.qlist;
    a.nwork = sl.qlist ? sl.nwork : nq;
    a.state = sl.state;
    a.st_d = sl.st_d;
    a.st_i = sl.st_i;
    a.step_budget = sl.step_budget;
    a.probe_step = sl.probe_step;
    a.probe_m = sl.probe_m;
    a.probe_f = sl.probe_f;
    nq = a.nwork;
    a.bcap = cfg.beam;
    a.lds_per_wave = wave_lds_bytes(cfg.beam, cfg.cache_slots, beam_key_bytes<D>());
    const int waves = cfg.waves;
    const size_t shmem = (size_t)a.lds_per_wave * waves;
    auto kern = k_beam<DTYPE, CPL, G>;
    int per_cu = 0;
    hipError_t e = kernel_occupancy((const void *)kern, waves * 64, shmem, &per_cu);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    int64_t blocks = (int64_t)per_cu * num_cus;
    const int64_t need = (nq + waves - 1) / waves;
    if (blocks > need) blocks = need;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(waves * 64), shmem, s, a);
    return hipGetLastError();
}

template <int DTYPE, int CPL, int G>
static hipError_t run_greedy(const DevIndex &ix, const SearchCfg &cfg, SearchBufs &sb,
                             int num_cus, hipStream_t s, hipEvent_t after_kernel) {
    using D = typename DistOf<DTYPE>::T;
    GreedyArgs a;
    a.ix = ix;
    a.cfg = cfg;
    a.sb = sb;
    using O = typename DistOf<DTYPE>::O;
    auto kern = k_greedy<DTYPE, CPL, G>;
    constexpr int GW = greedy_waves<DTYPE, CPL>();
    const size_t shmem = sizeof(GreedyLds<D, O, GW>);
    int per_cu = 0;
    hipError_t e = kernel_occupancy((const void *)kern, GW * 64, shmem, &per_cu);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    if (per_cu > 2) per_cu = 2;
    if (sb.local_grid > 0) {
        auto lk = k_greedy_local<DTYPE, CPL, G>;
        constexpr int LW = local_waves<DTYPE, CPL>();
        const size_t lsm = local_lds(sb.bm_words, sb.local_cap, LW, dapprox(DTYPE));
        int n = 0;
        e = kernel_occupancy((const void *)lk, LW * 64, lsm, &n);
        if (e != hipSuccess) return e;
        if (n < 1) return hipErrorInvalidConfiguration;
        const int lg = (int)std::min<int64_t>(sb.local_grid, (int64_t)n * num_cus);
        a.busy = local_busy(sb.local_full, lg, num_cus, !dfloat(DTYPE));
        hipLaunchKernelGGL(lk, dim3(lg), dim3(LW * 64), lsm, s, a);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // the level barriers need every workgroup resident: a cooperative launch
    dim3 grid((unsigned)(per_cu * num_cus)), block(GW * 64);
    void *args[] = {&a};
    e = hipLaunchCooperativeKernel((const void *)kern, grid, block, args, shmem, s);
    if (e != hipSuccess) return e;
    if (after_kernel) {
        e = hipEventRecord(after_kernel, s);
        if (e != hipSuccess) return e;
    }
    return launch_finalize(ix.dtype, sb, num_cus, s);
}

template <int DTYPE, int CPL, int G>
static hipError_t run_doubling(const DevIndex &ix, int64_t nq, const SearchCfg &cfg,
                               SearchBufs &sb, void *s_pool, int64_t s_cap, int num_cus,
                               hipStream_t s, int64_t *waves_total) {
    using D = typename DistOf<DTYPE>::T;
    DoublingArgs a;
    a.ix = ix;
    a.cfg = cfg;
    a.sb = sb;
    a.nq = nq;
    a.bcap = cfg.bcap;
    a.lds_per_wave = wave_lds_bytes(cfg.bcap, cfg.cache_slots, beam_key_bytes<D>());
    a.s_pool = (uint8_t *)s_pool;
    a.s_cap = s_cap;
    const int waves = cfg.waves;
    const size_t shmem = (size_t)a.lds_per_wave * waves;
    auto kern = k_doubling<DTYPE, CPL, G>;
    int per_cu = 0;
    hipError_t e = kernel_occupancy((const void *)kern, waves * 64, shmem, &per_cu);
    if (e != hipSuccess) return e;
    if (per_cu < 1) return hipErrorInvalidConfiguration;
    int64_t blocks = (int64_t)per_cu * num_cus;
    const int64_t need = (nq + waves - 1) / waves;
    if (blocks > need) blocks = need;
    if (blocks < 1) blocks = 1;
    if (waves_total) {
        // sizing call: report the grid, launch nothing
        *waves_total = blocks * waves;
        return hipSuccess;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(waves * 64), shmem, s, a);
    return hipGetLastError();
}

// waves_total != nullptr: only report how many waves the launch will use (the
// size of the per-wave S regions); otherwise launch with that many waves.

// (CPL, G) row splits the kernels are instantiated for: rows of 64 * 2^k and
// 192 * 2^k bytes up to 6144 bytes
#define RR_SPLITS(X) X(1, 4) X(1, 8) X(1, 16) X(1, 32) X(1, 64) X(2, 64) X(4, 64) \
    X(3, 4) X(3, 8) X(3, 16) X(3, 32) X(3, 64) X(6, 64)

// per data type: launch the kernel instantiated for the index's row split
template <int DTYPE>
hipError_t dispatch_beam_dt(const DevIndex &ix, int64_t nq, const SearchCfg &cfg, SearchBufs &sb,
                            int num_cus, hipStream_t s, const SlotArgs &sl, int cpl, int g) {
#define X(C, GG)                                                                              \
    if (cpl == C && g == GG) return run_beam<DTYPE, C, GG>(ix, nq, cfg, sb, num_cus, s, sl);
    RR_SPLITS(X)
#undef X
    return hipErrorInvalidValue;
}

template <int DTYPE>
hipError_t dispatch_greedy_dt(const DevIndex &ix, const SearchCfg &cfg, SearchBufs &sb,
                              int num_cus, hipStream_t s, hipEvent_t after_kernel, int cpl, int g) {
#define X(C, GG)                                                                              \
    if (cpl == C && g == GG) return run_greedy<DTYPE, C, GG>(ix, cfg, sb, num_cus, s, after_kernel);
    RR_SPLITS(X)
#undef X
    return hipErrorInvalidValue;
}

template <int DTYPE>
hipError_t dispatch_doubling_dt(const DevIndex &ix, int64_t nq, const SearchCfg &cfg,
                                SearchBufs &sb, void *s_pool, int64_t s_cap, int num_cus,
                                hipStream_t s, int64_t *waves_total, int cpl, int g) {
#define X(C, GG)                                                                              \
    if (cpl == C && g == GG)                                                                  \
        return run_doubling<DTYPE, C, GG>(ix, nq, cfg, sb, s_pool, s_cap, num_cus, s, waves_total);
    RR_SPLITS(X)
#undef X
    return hipErrorInvalidValue;
}

// Explicit instantiations live in rr_inst.hip, compiled once per data type
// (the search kernels of each type in a translation unit of their own).
#define RR_DECLARE_BEAM_GREEDY(DT, EXT)                                                        \
    EXT template hipError_t dispatch_beam_dt<DT>(const DevIndex &, int64_t, const SearchCfg &,  \
                                                 SearchBufs &, int, hipStream_t,               \
                                                 const SlotArgs &, int, int);                  \
    EXT template hipError_t dispatch_greedy_dt<DT>(const DevIndex &, const SearchCfg &,         \
                                                   SearchBufs &, int, hipStream_t, hipEvent_t, \
                                                   int, int);
#define RR_DECLARE_DOUBLING(DT, EXT)                                                           \
    EXT template hipError_t dispatch_doubling_dt<DT>(const DevIndex &, int64_t,                 \
                                                     const SearchCfg &, SearchBufs &, void *,  \
                                                     int64_t, int, hipStream_t, int64_t *,     \
                                                     int, int);

} // namespace rr
