// How the sort by cell cuts its keys into digits, its input into tiles and its scratch into arrays (host code alone,
// so that a host program can walk every key width).
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>

namespace anf {

constexpr int kPartBits = 8;                  // most bits of the leading digit, but for the longest keys
constexpr int kMaxBuckets = 1 << 9;           // nine bits where eight leave more than two digits: 31-bit keys, large calls
constexpr int kLastBits = 12;                 // most bits of a digit inside a bucket
constexpr int kLastBitsBig = 11;              // the same in large calls (sixteen waves' counts in LDS)

constexpr int kScanTile = 4096;               // elements per workgroup of a scan

// Buckets of the partitioned order and the tiles they are cut into: bucket b is slots [start[b], start[b + 1]) and
// tiles [tile[b], tile[b + 1]); an empty bucket has one (empty) tile.  The tiles of a bucket are grouped into the runs
// [run[b], run[b + 1]) that one workgroup of the digit sums walks each.
struct Buckets {
    uint32_t start[kMaxBuckets + 1];
    int32_t tile[kMaxBuckets + 1];
    int32_t run[kMaxBuckets + 1];
    int32_t done[kMaxBuckets];   // runs of the bucket summed so far, 0 between digits
};

// Tiles: 4096 elements in large calls, four to a thread, so that two workgroups of sixteen waves fit a CU (build of
// the clustered box of 16.7 million particles: 607 us; 512 threads with eight elements 672, with sixteen 767); fewer
// in small ones, which would leave most of the chip without a workgroup.
constexpr int kBigThreads = 1024, kBigItems = 4;
inline int tile_class(int64_t n) { return n <= 65536 ? 0 : (n <= (1 << 19) ? 1 : 2); }
inline int tile_size(int64_t n) {
    return tile_class(n) == 0 ? 1024 : (tile_class(n) == 1 ? 2048 : kBigThreads * kBigItems);
}
inline int64_t tile_number(int64_t n) { return (n + tile_size(n) - 1) / tile_size(n); }

// Log2 of the tiles in a run: 128, and more where the runs of one bucket that holds all tiles would be more than twice
// that.  Particles that crowd into one bucket (a zoomed box, one heavy cell) would leave its sums to one workgroup: 0.35
// to 1.2 ms a digit for 33.5 million particles, 25 to 50 us in runs.
inline int run_shift(int64_t n) {
    int s = 7;
    while (((int64_t)2 << (2 * s)) < tile_number(n)) s++;
    return s;
}

// Digits of a key of `bits` bits: `part` leading bits (0: one bucket), `mid` low bits (0: no middle scatter), `last`.
struct SortPlan {
    int part, mid, last;
};

// One bucket in small calls while its digit counts stay small (half a MB; with 2 MB they took 43 of 84 us), and where
// one digit of up to eight bits is the whole key (a box of 5^3 cells, 33.5 million particles: 579 us, 859 with a
// partition); else half of the bits up to eight lead (nine where eight would leave more than two digits), and what remains is
// one digit of at most twelve bits or two.
constexpr int64_t kOneBucketCounts = 1 << 17;
inline SortPlan sort_plan(int64_t n, int bits) {
    if (bits <= kPartBits ||
        (bits <= kLastBits && tile_class(n) < 2 && (tile_number(n) << bits) <= kOneBucketCounts))
        return SortPlan{0, 0, bits};
    const int most = tile_class(n) < 2 ? kLastBits : kLastBitsBig;
    const int part = std::max(std::min(kPartBits, (bits + 1) / 2), bits - 2 * most), rest = bits - part;
    if (rest <= most) return SortPlan{part, 0, rest};
    return SortPlan{part, rest / 2, rest - rest / 2};
}

inline size_t aligned(size_t bytes) { return (bytes + 255) & ~(size_t)255; }

// Scratch of the levels of a scan of n elements.
inline size_t scan_levels_bytes(int64_t n, size_t elem) {
    size_t bytes = 0;
    while (n > kScanTile) {
        int64_t nt = (n + kScanTile - 1) / kScanTile;
        bytes += 2 * (size_t)nt * elem + 256;
        n = nt;
    }
    return bytes;
}

// Scratch of one call: the buckets, the first slots of the digits in every run, and the digit counts of the tiles; the
// partition's counts, their sums and the scan's levels share the space of the latter.
struct SortScratch {
    size_t dbase, rows, total;   // offsets in bytes (the buckets are at 0), and the end
};

inline SortScratch sort_scratch(int64_t n, const SortPlan &pl) {
    const int64_t tiles = tile_number(n), nb = (int64_t)1 << pl.part;
    const int digit = std::max(pl.mid, pl.last);
    const int64_t rows = pl.part ? tiles + nb : tiles, runs = (tiles >> run_shift(n)) + nb;
    SortScratch s;
    s.dbase = aligned(sizeof(Buckets));
    s.rows = s.dbase + aligned((size_t)(sizeof(uint32_t) * runs) << digit);
    size_t bytes = (size_t)(sizeof(uint32_t) * rows) << digit;
    if (pl.part)
        bytes = std::max(bytes, 2 * (size_t)(nb * tiles) * sizeof(uint32_t) + 256 +
                                    scan_levels_bytes(nb * tiles, sizeof(uint32_t)));
    s.total = s.rows + aligned(bytes);
    return s;
}

// Enough for every call of at most n particles and keys of at most `bits` bits.
inline size_t sort_temp_bytes(int64_t n, int bits) {
    // small calls of one bucket: more particles can mean less scratch, so their bound stands for all of them
    size_t most = aligned(sizeof(Buckets)) + aligned(4 * sizeof(uint32_t) << std::min(bits, kLastBits)) +
                  kOneBucketCounts * sizeof(uint32_t);
    for (int b = 0; b <= bits; b++)
        for (int64_t m : {std::min<int64_t>(n, 65536), std::min<int64_t>(n, 1 << 19), n})
            most = std::max(most, sort_scratch(m, sort_plan(m, b)).total);
    return most;
}

}  // namespace anf
