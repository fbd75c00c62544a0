// rr_plan.h -- sizes that the host plans and the kernels rely on.  Plain C++,
// so that tests of these rules compile it for the CPU alone.
#pragma once

#include <cstddef>
#include <cstdint>

namespace rr {

// LDS of one wave of the beam and doubling kernels: scratch keys, the beam's
// array of bcap keys, the seen cache of cs ids.  A key takes key_bytes (8, or
// 12 for FP64 distances).  The scratch holds 64 keys, or 64-bit words with one
// bit for every key of the array (WaveBeam::merge_side).
constexpr int32_t beam_scratch_keys(int32_t bcap) { return bcap > 4096 ? (bcap + 63) / 64 : 64; }
constexpr int32_t wave_lds_bytes(int32_t bcap, int32_t cs, int32_t key_bytes) {
    return (((bcap + beam_scratch_keys(bcap)) * key_bytes + 15) & ~15) + cs * 4;
}

// What a search is admitted by, never less than wave_lds_bytes.  For doubling
// it counts the beam twice, more than the kernel holds: the widths that are
// taken, and the waves of a workgroup, follow from it.
constexpr size_t LDS_PER_CU = 160 * 1024;
constexpr size_t search_lds_bytes(bool doubling, int64_t bcap, int32_t cs, int32_t key_bytes) {
    return (size_t)(doubling ? 2 : 1) * key_bytes * bcap + 64 * 12 + cs * 4 + 128;
}

// doubling: the widest round is the first beam * 2^k >= max_beam
constexpr int64_t doubling_width(int64_t beam, int64_t max_beam) {
    int64_t b = beam;
    while (b < max_beam && b < (1 << 20)) b *= 2;
    return b;
}

// The list of a task inside one workgroup (k_greedy_local) is stopped this far
// from its end.  `open`: seeds that are not finished, drawn or not, read before
// the wave adds its points.  Let P be the end of the last addition that did not
// stop the list.  After P a wave adds the neighbours of the point it is at, 64 at
// most, and with that it stops the list itself; from then on it expands seeds
// only, and these were all open when P's wave read the count.  So the list ends
// at P + 64 (waves + open) at most.
constexpr int local_margin(int waves, int open) { return (waves + open) * 64; }
constexpr int LOCAL_SEEDS = 32;   // tasks with more seeds start in the level kernel
constexpr int LOCAL_WAVES = 16;   // waves of a workgroup at most
constexpr int LOCAL_LIST = 8192;  // found points a workgroup can hold at most
// the shortest list worth its start
constexpr int LOCAL_LEAST = local_margin(LOCAL_WAVES, LOCAL_SEEDS) + 256;

// How the dense scans split the base: `chunk` tiles a workgroup, and workgroup
// lin takes the chunk lin % x + x (lin / x / qblocks) for the query block
// lin / x % qblocks, x = 2^xcd_bits.  Workgroups are dealt to the 8 XCDs in turn,
// so with x = 8 all the query blocks of a chunk meet in one L2, and an XCD's
// share is its ceil(chunks / 8) chunks, however many query blocks there are.
// About SCAN_GROUPS workgroups, or of the splits into multiples of 8 the one
// with the smallest share; where even that is a twelfth or more above the mean
// (a base of few tiles, which any L2 holds), workgroups go to the XCDs as they
// come.
constexpr int64_t SCAN_GROUPS = 4096; // several times what is resident
struct ScanSplit {
    int64_t chunk, chunks; // tiles a workgroup, chunks
    int32_t xcd_bits;
    constexpr int64_t groups(int64_t qblocks) const {
        return qblocks * ((chunks + (1 << xcd_bits) - 1) >> xcd_bits << xcd_bits);
    }
};
constexpr ScanSplit scan_split(int64_t tiles, int64_t qblocks) {
    const int64_t want = SCAN_GROUPS / qblocks > 1 ? SCAN_GROUPS / qblocks : 1;
    int64_t chunk = (tiles + want - 1) / want, best = ((tiles + chunk - 1) / chunk + 7) / 8 * chunk;
    for (int64_t p = (want + 7) / 8 * 8; p >= 8; p -= 8) {
        const int64_t c = (tiles + p - 1) / p, share = ((tiles + c - 1) / c + 7) / 8 * c;
        // (not for the sake of 3%: fewer and longer chunks end less evenly)
        if (share * 33 < best * 32) {
            best = share;
            chunk = c;
        }
    }
    if (best * 8 * 12 < tiles * 13) return {chunk, (tiles + chunk - 1) / chunk, 3};
    chunk = (tiles + want - 1) / want;
    return {chunk, (tiles + chunk - 1) / chunk, 0};
}

} // namespace rr
