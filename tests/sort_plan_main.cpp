// Prints how the sort by cell plans calls, for the host-side test of its limits: first the limits, then one line per
// (n, key bits) with the tile size, the digits, the scratch of the call, the scratch a handle of that size
// holds, and the tiles of a run of the digit sums.
#include <cstdio>

#include "../paper_2110_11398_amd/csrc/sort_plan.h"

int main() {
    using namespace anf;
    printf("%d %d %d %zu\n", kMaxBuckets, kLastBits, kLastBitsBig, sizeof(Buckets));
    const int64_t sizes[] = {1,     1000,   1024,    1025,    20000,   32768,    32769,      65536,          65537,
                             70001, 131072, 200000,  262144,  262145,  524288,   524289,     600001,         4194304,
                             4194305, 33554432, 134217728, 1073741824, 2147483646};
    for (int64_t n : sizes)
        for (int bits = 5; bits <= 31; bits++) {
            const SortPlan p = sort_plan(n, bits);
            const SortScratch s = sort_scratch(n, p);
            printf("%lld %d %d %d %d %d %zu %zu %zu %zu %d\n", (long long)n, bits, tile_size(n), p.part, p.mid, p.last,
                   s.dbase, s.rows, s.total, sort_temp_bytes(n, bits), 1 << run_shift(n));
        }
    return 0;
}
