// Host driver for tests/test_plan.py: the sizes of rr_plan.h over all the
// values that the library accepts.  Prints what is wrong; exit status 1 then.
// Test infrastructure only.
//
// usage: plan_driver lds | list | list-drawn | scan
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>

#include "rr_plan.h"

using namespace rr;

static int bad = 0;
#define EXPECT(c, ...)                                                                        \
    do {                                                                                      \
        if (!(c) && ++bad <= 20) std::printf(__VA_ARGS__);                                    \
    } while (0)

// every (beam, widest round) that prepare_search takes: merge_side keeps a bit
// per key of a full beam in the scratch, and the kernels' LDS is what the
// search was admitted by
static long lds() {
    long seen = 0;
    for (int key = 8; key <= 12; key += 4)
        for (int cs = 64; cs <= 16384; cs *= 2)
            for (int beam = 1; beam <= 4096; ++beam)
                for (long b = beam, k = 0; b < (1 << 20); b *= 2, ++k) {
                    const bool doubling = k > 0;
                    if (doubling) EXPECT(doubling_width(beam, b) == b, "width %d..%ld\n", beam, b);
                    if (search_lds_bytes(doubling, b, cs, key) > LDS_PER_CU) break;
                    ++seen;
                    EXPECT(beam_scratch_keys((int)b) >= 64 && (b + 63) / 64 <= beam_scratch_keys((int)b),
                           "beam %d, round of %ld keys: %ld words of places in a scratch of %d\n", beam, b,
                           (b + 63) / 64, beam_scratch_keys((int)b));
                    EXPECT((size_t)wave_lds_bytes((int)b, cs, key) <= search_lds_bytes(doubling, b, cs, key),
                           "beam %d, round of %ld keys, %d slots: more LDS than admitted\n", beam, b, cs);
                }
    return seen;
}

// The list of k_greedy_local: its waves as step machines (every step one access
// of the shared counters), run in random orders in which some waves stall for
// long, with up to 64 points found at each expansion.  No list may pass its
// capacity, and every task ends.  `drawn`: the margin counts the seeds whose
// tickets are not drawn yet (a wave draws its next ticket before it adds the
// points it found), which the orders must be able to tell.
static long list(bool drawn) {
    std::mt19937 g(5);
    long seen = 0, over = 0;
    for (int run = 0; run < 800; ++run) {
        const int GW = 1 + (int)(g() % LOCAL_WAVES), nseed = (int)(g() % (LOCAL_SEEDS + 1));
        const int cap = LOCAL_LEAST + (run % 3 ? 0 : (int)(g() % (LOCAL_LIST - LOCAL_LEAST))) / 4 * 4;
        int head = 0, tail = 0, done = 0, seeds = 0, top = 0;
        bool stop = false;
        std::vector<char> there(cap + 128 * LOCAL_WAVES, 0);
        struct W { int pc = 0, i = 0, ni = 0, m = 0, pos = 0, open = 0, stall = 0; };
        std::vector<W> w(GW);
        // waves that stall, and where: before they add the points of a seed
        const int slow = (int)(g() % (GW + 1)), few = (int)(g() % 4);
        for (auto &x : w) x.i = head++;
        int left = GW, steps = 0;
        for (; left > 0 && steps < 4000000; ++steps) {
            const int k = (int)(g() % GW);
            W &x = w[k];
            if (x.pc == 6 || (x.stall > 0 && x.stall--)) continue;
            switch (x.pc) {
            case 0: // the ticket's point
                if (x.i < nseed) { x.pc = 1; break; }
                if (stop) { x.pc = 6; --left; break; }
                if (x.i - nseed < tail && there[x.i - nseed]) { x.pc = 1; break; }
                if (done == nseed + tail) { x.pc = 6; --left; }
                break;
            case 1: // the next ticket, then the neighbours
                x.ni = head++;
                x.m = few ? 64 : (int)(g() % 65);
                x.pc = 2;
                if (k < slow && x.i < nseed) x.stall = 20000;
                break;
            case 2:
                x.open = nseed - seeds;
                x.pc = 3;
                break;
            case 3:
                x.pos = tail;
                tail += x.m;
                x.pc = 4;
                if (g() % 8 == 0) x.stall = (int)(g() % 400);
                break;
            case 4:
                if (drawn) x.open = std::max(0, nseed - head);
                if (x.m && x.pos + x.m > cap - local_margin(GW, x.open)) stop = true;
                for (int j = 0; j < x.m && x.pos + j < (int)there.size(); ++j) there[x.pos + j] = 1;
                top = std::max(top, x.pos + x.m);
                x.pc = 5;
                break;
            default: // finished
                if (x.i < nseed) ++seeds;
                ++done;
                x.i = x.ni;
                x.pc = 0;
            }
        }
        ++seen;
        over += top > cap;
        EXPECT(top <= cap, "waves %d seeds %d: %d points in a list of %d\n", GW, nseed, top, cap);
        EXPECT(left == 0, "waves %d seeds %d: not ended\n", GW, nseed);
    }
    std::printf("%ld lists passed their capacity\n", over);
    return seen;
}

// Dense scans: every tile of the base is taken once for every query block, and
// no XCD has much more than the mean of the tiles (workgroup i runs on XCD i % 8)
static long scan() {
    long seen = 0;
    std::vector<long> tiles = {1, 2, 7, 8, 9, 15, 16, 17, 63, 64, 65, 79, 100, 157, 782, 1000, 7813, 15625, 70313};
    std::mt19937 g(9);
    for (int i = 0; i < 300; ++i) tiles.push_back(1 + (long)(g() % (i < 150 ? 300 : 20000)));
    for (long t : tiles)
        for (long qb : {1l, 2l, 3l, 20l, 79l, 98l, 205l, 313l, 391l, 400l, 586l, 800l, 1954l, 7813l}) {
            const ScanSplit s = scan_split(t, qb);
            ++seen;
            EXPECT(s.chunk >= 1 && s.chunks * s.chunk >= t && (s.chunks - 1) * s.chunk < t && (s.xcd_bits == 0 || s.xcd_bits == 3),
                   "%ld tiles, %ld query blocks: chunks %ld of %ld\n", t, qb, (long)s.chunks, (long)s.chunk);
            double load[8] = {0}, most = 0, all = 0;
            std::vector<char> taken;
            if (t * qb < 200000) taken.assign(t * qb, 0);
            for (long lin = 0; lin < s.groups(qb); ++lin) {
                const long x = 1l << s.xcd_bits, p = lin % x + x * (lin / x / qb), q = lin / x % qb;
                const long t0 = p * s.chunk, t1 = std::min<long>(t, t0 + s.chunk);
                for (long k = t0; k < t1 && !taken.empty(); ++k) ++taken[k * qb + q];
                if (t1 > t0) load[lin % 8] += t1 - t0;
            }
            for (double l : load) most = std::max(most, l), all += l;
            EXPECT(all == (double)t * qb && std::all_of(taken.begin(), taken.end(), [](char c) { return c == 1; }),
                   "%ld tiles, %ld query blocks: not every tile once\n", t, qb);
            // (a last chunk for itself when workgroups are few)
            EXPECT(most <= 1.1 * all / 8 + 2 * s.chunk, "%ld tiles, %ld query blocks: %g tiles on one XCD of %g\n", t, qb,
                   most, all / 8);
        }
    return seen;
}

int main(int argc, char **argv) {
    long seen = 0;
    if (argc > 1 && !std::strcmp(argv[1], "lds")) seen = lds();
    if (argc > 1 && !std::strcmp(argv[1], "list")) seen = list(false);
    if (argc > 1 && !std::strcmp(argv[1], "scan")) seen = scan();
    if (argc > 1 && !std::strcmp(argv[1], "list-drawn")) seen = list(true);
    std::printf("%ld checked, %d wrong\n", seen, bad);
    return bad || !seen;
}
