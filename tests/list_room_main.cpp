// Prints the lists the force pass holds for batches of boxes, for the host-side test: one line per batch with the
// particles, the cells, slots and items of the lists, those the boxes' rooms add up to, and the least lists; then one
// line per pair count and sinks per lane with the least length of a source part.
#include <cstdio>
#include <vector>

#include "../paper_2110_11398_amd/csrc/nf_internal.h"

struct Run {
    long long boxes, n, K;
};

int main() {
    const std::vector<std::vector<Run>> batches = {
        {{1, 1, 5}}, {{1, 13824, 8}}, {{1, 131072, 16}}, {{1, 2147483646, 256}}, {{1, 200000000, 1290}},
        {{1000, 131072, 16}}, {{2100, 131072, 16}}, {{2000, 110592, 14}}, {{4096, 500, 5}}, {{65536, 100, 3}},
        {{65536, 32767, 20}}, {{48, 32768, 9}}, {{64, 65536, 12}}, {{64, 2560000, 100}},
        {{5, 0, 3}, {1, 100000000, 300}, {500, 70000, 11}, {3, 0, 7}, {1, 1, 3}}};
    for (const auto &batch : batches) {
        long long n = 0, cells = 0, boxes = 0, slots = 0, items = 0;
        for (const Run &r : batch) {
            n += r.boxes * r.n;
            cells += r.boxes * r.K * r.K * r.K;
            boxes += r.boxes;
            slots += r.boxes * anf::box_slots(r.n);
            items += r.boxes * anf::box_items(r.n, r.K * r.K * r.K);
        }
        const anf::ListRoom r = anf::list_room(n, cells, boxes), l = anf::least_room(n, cells);
        printf("%lld %lld %lld %lld %lld %lld %lld %lld %lld\n", boxes, n, cells, (long long)r.slots,
               (long long)r.items, slots, items, (long long)l.slots, (long long)l.items);
    }
    printf("\n");
    for (int S : {1, 2, 4})
        for (unsigned long long pairs = 0; pairs < (1ull << 45); pairs = 2 * pairs + 1234567)
            printf("%d %llu %lld\n", S, pairs, anf::least_part(pairs, S));
    return 0;
}
