// rr_scan.h -- what the dense scans of rr_scan.hip and rr_scan_f32.hip share.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rr_internal.h"

namespace rr {

enum { SCAN_NN = 0, SCAN_RANGE = 1 };

struct ScanArgs {
    DevIndex ix;
    const uint8_t *qpad;  // [nq][row_bytes]
    const QThresh *qth;   // [nq] (range mode)
    int64_t nq;
    int64_t chunk;        // base points per workgroup
    int32_t qblocks;      // query blocks (integer range scan, split scan)
    int32_t xcd_bits;     // of scan_split
    // nn mode
    unsigned long long *nn_bits; // [nq] min distance bits (uint32 value or double bits)
    // range mode: hits appended as items (task = query)
    unsigned long long *item_key; // (query << 32) | id
    void *item_dist;
    int64_t item_cap;
    unsigned long long *item_cursor;
    unsigned long long *task_cnt;
    unsigned long long *overflow;
};

// the workgroup's chunk of the base and its query block (scan_split)
struct ScanPlace {
    int64_t chunk;
    int qblock;
};
__device__ __forceinline__ ScanPlace scan_place(const ScanArgs &a) {
    const uint32_t lin = blockIdx.x >> a.xcd_bits, x = blockIdx.x & ((1u << a.xcd_bits) - 1u), n = a.qblocks;
    // (uniform, which the compiler does not see behind a division: with the
    // chunk's bounds in vector registers the integer range scan took 3% longer)
    return {__builtin_amdgcn_readfirstlane((int)(x + ((lin / n) << a.xcd_bits))),
            __builtin_amdgcn_readfirstlane((int)(lin % n))};
}

// order-preserving map of a double to an unsigned key (atomicMin over
// signed distances) and back
__device__ __forceinline__ unsigned long long dbl_order(double d) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(d);
    return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double dbl_unorder(unsigned long long k) {
    return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}

// rr_scan_f32.hip: whether the split-bfloat16 scan takes this index, and its
// two scans (ws: scan_ws_bytes, 16-byte aligned)
bool scan_split_ok(const DevIndex &ix);
// the range scan, but for the tiles that a list in ws names (their count goes to
// item_cursor[1]); the second call decides those
hipError_t launch_split_range(const ScanArgs &a, uint8_t *ws, hipStream_t s);
hipError_t launch_split_range_dense(const ScanArgs &a, uint8_t *ws, hipStream_t s);
// writes nn_bits (dbl_order of the smallest distance of every query)
hipError_t launch_split_nn(const ScanArgs &a, uint8_t *ws, hipStream_t s);

} // namespace rr
