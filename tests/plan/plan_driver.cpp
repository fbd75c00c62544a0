// Host driver for tests/test_plan.py: the sizes of rr_plan.h over all the
// values that the library accepts.  Prints what is wrong; exit status 1 then.
// Test infrastructure only.
//
// usage: plan_driver lds
#include <cstdio>
#include <cstring>

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

int main(int argc, char **argv) {
    long seen = 0;
    if (argc > 1 && !std::strcmp(argv[1], "lds")) seen = lds();
    std::printf("%ld checked, %d wrong\n", seen, bad);
    return bad || !seen;
}
