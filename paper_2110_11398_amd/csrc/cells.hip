// Cell construction for the near-field force: binning, a stable sort of the
// particles by cell, the cell offsets, and the cell-relative FP32 layout.
//
// Sec. 3.1 of the paper cuts each periodic box into a cubic lattice of CPD^3
// cells; the near field of a particle is defined by the cells around its own.
// The paper's CPU pipeline re-bins particles and transposes positions for the
// GPU every step (Table "tbl:timing": "Transpose Positions", "Merge New
// Particles").  Here the equivalent is done on the device, in HBM:
//
//   k_bin          cell of every particle (FP64 cell rule) and a tile histogram of its leading digit
//   k_seg_scatter  as partition: stable scatter by the leading digit (up to 8 bits) of coordinates, input index and
//                  cell; every later step then works inside one bucket, whose few MB stay in cache
//   k_seg_hist,    per bucket: digit counts of every tile, their exclusive sums over runs of tiles, and the first slots
//   k_seg_sums     of the digits in every run (k_seg_base where one bucket has several runs)
//   k_seg_scatter  stable scatter inside the buckets; the last one writes the sorted keys, the permutation and
//                  the cell-relative coordinates in cell widths, FP64 -> FP32
//
// Where the last digit spans the whole cell index inside a bucket (keys of up to 19 bits in large calls), its sums
// are the cell offsets; longer keys take one more digit before it, and k_run_ends with a max-scan the offsets.
// Small calls and boxes of few cells skip the partition: one bucket, one digit.
//
// Bound by memory: coordinates move in order three times (44 bytes read and 44 written per particle with the keys),
// against one random 12-byte gather, a cache line each, when only keys and indices were sorted.  Clustered box of
// 16.7 million particles in random order 866 -> 610 us, late-time box of 33.5 million 1960 -> 1570, 6 million 358 ->
// 200, 2 million 154 -> 91.
//
// Every step is deterministic: particles of a cell stay in input order.
#include <algorithm>
#include <climits>
#include <cstring>

#include "nf_internal.h"
#include "sort_plan.h"

namespace anf {

namespace {

constexpr int kTileThreads = 256;
constexpr int kTileItems = 16;
constexpr int kTile = kTileThreads * kTileItems;  // elements per workgroup of a scan
static_assert(kTile == kScanTile, "scratch of the scans");

inline unsigned grid_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// ---------------------------------------------------------------- fills / boxes

__global__ void k_fill_i32(int32_t *p, int64_t n, int32_t v) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

constexpr int kBoxChunk = 24;
struct BoxChunk {
    BoxDev b[kBoxChunk];
    int first, count;
};

__global__ void k_set_boxes(BoxChunk c, BoxDev *dst) {
    int i = threadIdx.x;
    if (i < c.count) dst[c.first + i] = c.b[i];
}

// The cell rule along one axis, every FP64 operation rounded on its own:
//   xt = x - L*floor(x/L),  t = xt*s (s = K/L),  c = min(floor(t), K-1).
__device__ inline int axis_cell(double x, double L, double s, int K, double *t_out) {
#pragma clang fp contract(off)
    // x / L rounds below 1 for x up to L (1 - 2^-50): floor is 0 and xt is x, without the division
    double xt = x;
    if (!(x >= 0.0 && x < L * (1.0 - 0x1p-50))) {
        double q = floor(x / L);
        xt = x - L * q;
    }
    double t = xt * s;
    double f = floor(t);
    int c = (f >= (double)(K - 1)) ? (K - 1) : (int)f;
    if (c < 0) c = 0;
    *t_out = t;
    return c;
}

// Cell of every particle of a tile, and the tile's histogram of bits [shift, shift + bits) of the cell index:
// row `tile` of hist when by_row, else column `tile` ([digit][tile], for one scan over all of it).
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_bin(const float *__restrict__ pos, int64_t n,
                                                 const BoxDev *__restrict__ boxes, int n_boxes,
                                                 int32_t *__restrict__ keys, int shift, int bits,
                                                 uint32_t *__restrict__ hist, int by_row, int *err) {
    extern __shared__ uint32_t smem_u32[];
    uint32_t *h = smem_u32;
    const int D = 1 << bits, tid = threadIdx.x;
    for (int d = tid; d < D; d += THREADS) h[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * (THREADS * ITEMS);
#pragma unroll 4
    for (int r = 0; r < ITEMS; r++) {
        const int64_t i = base + r * THREADS + tid;
        if (i >= n) break;
        const int b = n_boxes > 1 ? box_of_particle(boxes, n_boxes, i) : 0;
        const BoxDev B = boxes[b];
        const double x = pos[3 * i], y = pos[3 * i + 1], z = pos[3 * i + 2];
        int32_t key = B.cell_base;
        if (isfinite(x) && isfinite(y) && isfinite(z)) {
            double t;
            const int cx = axis_cell(x, B.L, B.s, B.K, &t);
            const int cy = axis_cell(y, B.L, B.s, B.K, &t);
            const int cz = axis_cell(z, B.L, B.s, B.K, &t);
            key = B.cell_base + (cx * B.K + cy) * B.K + cz;
        } else {
            atomicCAS(err, 0, ABACUS_NF_ENONFINITE);
        }
        keys[i] = key;
        atomicAdd(&h[((uint32_t)key >> shift) & (uint32_t)(D - 1)], 1u);
    }
    __syncthreads();
    for (int d = tid; d < D; d += THREADS) {
        if (by_row)
            hist[(int64_t)blockIdx.x * D + d] = h[d];
        else
            hist[(int64_t)d * gridDim.x + blockIdx.x] = h[d];
    }
}

// ---------------------------------------------------------------- scans

struct OpAdd {
    template <typename T> __device__ T operator()(T a, T b) const { return a + b; }
};
struct OpMax {
    template <typename T> __device__ T operator()(T a, T b) const { return a > b ? a : b; }
};

// Scan of one tile of kTile elements: each thread scans 16 consecutive
// elements, a Hillis-Steele pass over the 256 thread totals adds the prefix.
template <typename T, typename Op>
__global__ __launch_bounds__(kTileThreads) void k_scan_tile(const T *in, T *out, T *sums, int64_t n, int inclusive,
                                                           T identity) {
    __shared__ T s[kTileThreads];
    Op op;
    int tid = threadIdx.x;
    int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)tid * kTileItems;
    T v[kTileItems];
    T run = identity;
#pragma unroll
    for (int k = 0; k < kTileItems; k++) {
        int64_t i = base + k;
        T x = i < n ? in[i] : identity;
        T nr = op(run, x);
        v[k] = inclusive ? nr : run;
        run = nr;
    }
    s[tid] = run;
    __syncthreads();
    for (int off = 1; off < kTileThreads; off <<= 1) {
        T y = tid >= off ? s[tid - off] : identity;
        __syncthreads();
        s[tid] = op(s[tid], y);
        __syncthreads();
    }
    T prefix = tid > 0 ? s[tid - 1] : identity;
#pragma unroll
    for (int k = 0; k < kTileItems; k++) {
        int64_t i = base + k;
        if (i < n) out[i] = op(prefix, v[k]);
    }
    if (sums && tid == kTileThreads - 1) sums[blockIdx.x] = s[kTileThreads - 1];
}

template <typename T, typename Op>
__global__ void k_scan_add(T *out, const T *offs, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        int64_t b = i / kTile;
        if (b > 0) out[i] = Op()(offs[b], out[i]);
    }
}

template <typename T, typename Op>
hipError_t scan_impl(const T *in, T *out, int64_t n, bool inclusive, T identity, char *temp, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    int64_t nt = (n + kTile - 1) / kTile;
    if (nt == 1) {
        hipLaunchKernelGGL((k_scan_tile<T, Op>), dim3(1), dim3(kTileThreads), 0, st, in, out, (T *)nullptr, n,
                           (int)inclusive, identity);
        return hipGetLastError();
    }
    T *sums = (T *)temp;
    T *offs = sums + nt;
    char *next = (char *)(((uintptr_t)(offs + nt) + 255) & ~(uintptr_t)255);
    hipLaunchKernelGGL((k_scan_tile<T, Op>), dim3((unsigned)nt), dim3(kTileThreads), 0, st, in, out, sums, n,
                       (int)inclusive, identity);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = scan_impl<T, Op>(sums, offs, nt, false, identity, next, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_scan_add<T, Op>), dim3(grid_for(n, 256)), dim3(256), 0, st, out, offs, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------- sort by cell

__global__ __launch_bounds__(kMaxBuckets) void k_buckets(const uint32_t *__restrict__ toff, int ntiles, int nb, int64_t n,
                                                         int tile, int run_shift, Buckets *__restrict__ o) {
    __shared__ int32_t wsum[2][kMaxBuckets / 64];
    const int b = threadIdx.x, lane = b & 63;
    const uint32_t lo = b < nb ? toff[(int64_t)b * ntiles] : (uint32_t)n;
    const uint32_t hi = b + 1 < nb ? toff[(int64_t)(b + 1) * ntiles] : (uint32_t)n;
    const int t = b < nb ? (hi > lo ? (int)((hi - lo + tile - 1) / tile) : 1) : 0;
    const int r = (t + (1 << run_shift) - 1) >> run_shift;
    int tiles = t, runs = r;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(tiles, off), z = __shfl_up(runs, off);
        if (lane >= off) {
            tiles += y;
            runs += z;
        }
    }
    if (lane == 63) {
        wsum[0][b >> 6] = tiles;
        wsum[1][b >> 6] = runs;
    }
    __syncthreads();
    for (int w = 0; w < (b >> 6); w++) {
        tiles += wsum[0][w];
        runs += wsum[1][w];
    }
    o->start[b] = lo;
    o->tile[b] = tiles - t;
    o->run[b] = runs - r;
    o->done[b] = 0;
    if (b == kMaxBuckets - 1) {
        o->start[kMaxBuckets] = (uint32_t)n;
        o->tile[kMaxBuckets] = tiles;
        o->run[kMaxBuckets] = runs;
    }
}

// The last of the nb buckets whose first tile or run is at most g: the lanes of a wave look at four each at once (a
// binary search waits for eight or nine loads in turn).
__device__ inline int bucket_at(const int32_t *__restrict__ first, int nb, int g) {
    const int lane = threadIdx.x & 63;
    int count = 0;
    for (int i = 0; i < nb; i += 256) {
        int v[4];
#pragma unroll
        for (int q = 0; q < 4; q++) v[q] = i + 64 * q + lane < nb ? first[i + 64 * q + lane] : INT_MAX;
#pragma unroll
        for (int q = 0; q < 4; q++) count += __popcll(__ballot(v[q] <= g));
    }
    return count - 1;
}

// Run, first slot and number of slots of tile g (bk null: one bucket of n slots); false past the last tile.
__device__ inline bool seg_tile(const Buckets *__restrict__ bk, int nb, int64_t n, int tile, int run_shift, int g, int &run,
                                int64_t &base, int &count) {
    run = g >> run_shift;
    int64_t end = n;
    base = (int64_t)g * tile;
    if (bk) {
        if (g >= bk->tile[kMaxBuckets]) return false;
        const int b = bucket_at(bk->tile, nb, g), in = g - bk->tile[b];
        run = bk->run[b] + (in >> run_shift);
        base = (int64_t)bk->start[b] + (int64_t)in * tile;
        end = bk->start[b + 1];
    }
    const int64_t left = end - base;
    count = left < tile ? (left > 0 ? (int)left : 0) : tile;
    return true;
}

template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_seg_hist(const int32_t *__restrict__ keys, int64_t n,
                                                      const Buckets *__restrict__ bk, int nb, int shift, int bits,
                                                      uint32_t *__restrict__ rows) {
    extern __shared__ uint32_t smem_u32[];
    uint32_t *h = smem_u32;
    int run, count;
    int64_t base;
    if (!seg_tile(bk, nb, n, THREADS * ITEMS, 0, blockIdx.x, run, base, count)) return;
    const int D = 1 << bits, tid = threadIdx.x;
    for (int d = tid; d < D; d += THREADS) h[d] = 0;
    __syncthreads();
#pragma unroll 4
    for (int r = 0; r < ITEMS; r++) {
        const int i = r * THREADS + tid;
        if (i < count) atomicAdd(&h[((uint32_t)keys[base + i] >> shift) & (uint32_t)(D - 1)], 1u);
    }
    __syncthreads();
    for (int d = tid; d < D; d += THREADS) rows[(int64_t)blockIdx.x * D + d] = h[d];
}

__device__ inline void add4(uint4 &x, const uint4 &y) {
    x.x += y.x;
    x.y += y.y;
    x.z += y.z;
    x.w += y.w;
}

// Exclusive sums down a column of rows [t0, t1) of Q groups of four counts each, in place, the loads of eight rows in
// flight; returns the totals.
__device__ inline uint4 scan_rows(uint4 *col, int t0, int t1, int64_t Q) {
    uint4 run = make_uint4(0, 0, 0, 0);
    int t = t0;
    for (; t + 8 <= t1; t += 8, col += 8 * Q) {
        uint4 v[8];
#pragma unroll
        for (int q = 0; q < 8; q++) v[q] = col[q * Q];
#pragma unroll
        for (int q = 0; q < 8; q++) {
            col[q * Q] = run;
            add4(run, v[q]);
        }
    }
    for (; t < t1; t++, col += Q) {
        const uint4 v = *col;
        *col = run;
        add4(run, v);
    }
    return run;
}

// First slots of four digits of bucket b, from the digits' totals; with cell_start, bits that end the key: slot of
// every cell.  The whole workgroup.
constexpr int kSegScanThreads = 1 << (kLastBits - 2);
__device__ inline uint4 digit_starts(const uint4 &sum, int b, uint32_t start, int Q, int64_t n,
                                     int32_t *__restrict__ cell_start, int64_t n_cells) {
    __shared__ uint32_t wsum[kSegScanThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t s = sum.x + sum.y + sum.z + sum.w;
    uint32_t incl = s;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[tid >> 6] = incl;
    __syncthreads();
    uint32_t first = start + incl - s;
    for (int w = 0; w < (tid >> 6); w++) first += wsum[w];
    const uint4 o = make_uint4(first, first + sum.x, first + sum.x + sum.y, first + sum.x + sum.y + sum.z);
    if (cell_start && tid < Q) {
        const int64_t g = 4 * ((int64_t)b * Q + tid);
        const uint32_t v[4] = {o.x, o.y, o.z, o.w};
        for (int q = 0; q < 4; q++)
            if (g + q < n_cells) cell_start[g + q] = (int32_t)v[q];
    }
    if (cell_start && b == 0 && tid == 0) cell_start[n_cells] = (int32_t)n;
    return o;
}

// The totals of runs [r0, r1) of bucket b become the first slots of the digits in each run.  The whole workgroup.
__device__ inline void run_bases(uint32_t *dbase, int r0, int r1, int Q, int b, uint32_t start, int64_t n,
                                 int32_t *__restrict__ cell_start, int64_t n_cells) {
    const int tid = threadIdx.x;
    uint4 *col = (uint4 *)dbase + (int64_t)r0 * Q + tid;
    uint4 sum = make_uint4(0, 0, 0, 0);
    if (tid < Q) sum = scan_rows(col, r0, r1, Q);
    const uint4 first = digit_starts(sum, b, start, Q, n, cell_start, n_cells);
    if (tid < Q)
#pragma unroll 8
        for (int r = r0; r < r1; r++, col += Q) {
            uint4 v = *col;
            add4(v, first);
            *col = v;
        }
}

// One workgroup per run of tiles: their rows of digit counts become exclusive sums over the run, four digits to a
// thread, and dbase, per run, the digits' totals; then the first slots, by the run itself where it is its bucket's only
// one (`single`: every one is), else by the run of the bucket that ends last.  (A kernel of its own for the latter cost
// every call of more than 128 tiles 5 us a digit.)  With one bucket of several runs k_seg_base does it.
__global__ __launch_bounds__(kSegScanThreads) void k_seg_sums(uint32_t *rows, uint32_t *dbase, Buckets *bk, int nb, int64_t n,
                                                              int ntiles, int run_shift, int bits, int single,
                                                              int32_t *__restrict__ cell_start, int64_t n_cells) {
    __shared__ int last;
    const int Q = 1 << (bits - 2), tid = threadIdx.x, g = blockIdx.x;   // Q groups of four digits
    int b = 0, t0 = g << run_shift, end = ntiles, r0 = 0, r1 = single ? 1 : 2;
    uint32_t start = 0;
    if (bk) {
        if (g >= bk->run[kMaxBuckets]) return;
        b = single ? g : bucket_at(bk->run, nb, g);
        r0 = bk->run[b];
        r1 = bk->run[b + 1];
        t0 = bk->tile[b] + ((g - r0) << run_shift);
        end = bk->tile[b + 1];
        start = bk->start[b];
    }
    const int t1 = end - t0 < (1 << run_shift) ? end : t0 + (1 << run_shift);
    uint4 sum = make_uint4(0, 0, 0, 0);
    if (tid < Q) sum = scan_rows((uint4 *)rows + (int64_t)t0 * Q + tid, t0, t1, Q);
    if (r1 - r0 == 1) sum = digit_starts(sum, b, start, Q, n, cell_start, n_cells);
    if (tid < Q) ((uint4 *)dbase)[(int64_t)g * Q + tid] = sum;
    if (!bk || r1 - r0 == 1) return;
    // the totals of every run are in memory before it is counted, and read after the last count
    __threadfence();
    __syncthreads();
    if (tid == 0) {
        last = atomicAdd(&bk->done[b], 1) == r1 - r0 - 1;
        if (last) bk->done[b] = 0;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    run_bases(dbase, r0, r1, Q, b, start, n, cell_start, n_cells);
}

// The first slots of one bucket of several runs.
__global__ __launch_bounds__(kSegScanThreads) void k_seg_base(uint32_t *dbase, int64_t n, int nruns, int bits,
                                                              int32_t *__restrict__ cell_start, int64_t n_cells) {
    run_bases(dbase, 0, nruns, 1 << (bits - 2), 0, 0u, n, cell_start, n_cells);
}

// What a scatter reads and writes.
enum SegOut {
    kSegPart,      // positions by input index -> coordinates with their input index
    kSegMid,       // coordinates with their input index -> the same
    kSegLastPos,   // positions by input index -> the sorted layout
    kSegLast       // coordinates with their input index -> the sorted layout
};

struct SegArgs {
    const int32_t *kin;
    const float *pos;            // kSegPart, kSegLastPos
    const float4 *pay;           // kSegMid, kSegLast: x, y, z, input index (bits)
    const uint32_t *rows;        // per tile and digit: first slot among the run's (kSegPart: absolute, [digit][tile])
    const uint32_t *dbase;       // per run and digit: first slot
    const Buckets *bk;
    int nb;                      // buckets
    const BoxDev *boxes;
    int n_boxes;
    int64_t n;
    int shift, bits, run_shift;
    int32_t *kout;
    int32_t *vout;               // last scatter: permutation
    float4 *out;                 // coordinates, or spos in the last scatter
};

constexpr int kStageMost = 2048;   // elements staged in LDS at a time

// spos = (t_x - (c_x + 1/2), t_y - (c_y + 1/2), t_z - (c_z + 1/2), c_z) where t = xt*K/L is the wrapped
// coordinate in cell widths: positions relative to the centre of their own cell, in cell widths, rounded once to
// FP32.
__device__ inline float4 cell_relative(float px, float py, float pz, const BoxDev &B) {
    const double x = px, y = py, z = pz;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    if (isfinite(x) && isfinite(y) && isfinite(z)) {
        double tx, ty, tz;
        const int cx = axis_cell(x, B.L, B.s, B.K, &tx);
        const int cy = axis_cell(y, B.L, B.s, B.K, &ty);
        const int cz = axis_cell(z, B.L, B.s, B.K, &tz);
        o.x = (float)(tx - ((double)cx + 0.5));
        o.y = (float)(ty - ((double)cy + 0.5));
        o.z = (float)(tz - ((double)cz + 0.5));
        o.w = (float)cz;
    }
    return o;
}

// Stable scatter of one tile.  Wave w owns the contiguous span [w * 64 ITEMS, (w + 1) * 64 ITEMS) of the tile, read
// in ITEMS rounds of 64.  Within a round, lanes with equal digits are found with one ballot per digit bit; a lane's
// rank is the number of equal lanes below it plus the wave's running count of that digit.  Wave counts are then
// prefix-summed across the waves and the tile's digit totals across the digits: every element gets its position in
// the tile sorted by digit.  The elements wait in registers (read in order) and go through LDS in that order, 2048
// positions at a time, so that consecutive threads write consecutive elements of a run.  (With element numbers
// staged instead, and the elements read from the tile in sorted order, every lane touched a cache line of its own:
// 16.7 million particles 333 + 486 us for the two scatters.)
template <int THREADS, int ITEMS, int OUT>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(THREADS == 1024 ? 8 : 4))) void k_seg_scatter(SegArgs a) {
    constexpr int TILE = THREADS * ITEMS, WAVES = THREADS / 64, STAGE = TILE < kStageMost ? TILE : kStageMost;
    extern __shared__ __align__(16) uint32_t smem_u32[];
    const int D = 1 << a.bits;
    float4 *stage = (float4 *)smem_u32;                   // [STAGE] x, y, z, input index
    int32_t *skey = (int32_t *)(stage + STAGE);           // [STAGE]
    uint32_t *gd = (uint32_t *)(skey + STAGE);            // [D] global slot of a digit's run minus its tile position
    uint32_t *wsum = gd + D;                              // [WAVES]
    uint16_t *wcnt = (uint16_t *)(wsum + WAVES);          // [WAVES][D] counts, then tile positions
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    int run_of, count;
    int64_t base;
    if (!seg_tile(OUT == kSegPart || OUT == kSegLastPos ? nullptr : a.bk, a.nb, a.n, TILE, a.run_shift, blockIdx.x,
                           run_of, base, count))
        return;
    for (int d = tid; d < WAVES * D / 2; d += THREADS) ((uint32_t *)wcnt)[d] = 0;
    __syncthreads();
    const uint32_t mask = (uint32_t)(D - 1);
    const uint64_t below_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const uint32_t span = w * 64 * ITEMS + lane, un = (uint32_t)count;   // this thread's elements: span + 64 r
    const int32_t *kin = a.kin + base;
    uint32_t dig[ITEMS];   // digit, and the rank above it; then the position in the sorted tile
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const uint32_t i = span + r * 64;
        dig[r] = i < un ? ((uint32_t)kin[i] >> a.shift) & mask : 0u;
    }
    // the elements themselves: on their way while the ranks are formed
    constexpr bool kFromPos = OUT == kSegPart || OUT == kSegLastPos;
    float ex[ITEMS], ey[ITEMS], ez[ITEMS];
    int32_t ei[kFromPos ? 1 : ITEMS];
    const float *pos = kFromPos ? a.pos + 3 * base : nullptr;
    const float4 *pay = kFromPos ? nullptr : a.pay + base;
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const uint32_t i = span + r * 64;
        ex[r] = ey[r] = ez[r] = 0.f;
        if constexpr (!kFromPos) ei[r] = 0;
        if (i < un) {
            if constexpr (kFromPos) {
                ex[r] = pos[3 * i];
                ey[r] = pos[3 * i + 1];
                ez[r] = pos[3 * i + 2];
            } else {
                const float4 v = pay[i];
                ex[r] = v.x;
                ey[r] = v.y;
                ez[r] = v.z;
                ei[r] = __float_as_int(v.w);
            }
        }
    }
    uint16_t *wc = wcnt + w * D;
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        const bool valid = span + r * 64 < un;
        const uint32_t d = dig[r];
        uint64_t m = __ballot(valid);
        for (int b = 0; b < a.bits; b++) {
            const int bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const uint32_t below = (uint32_t)__popcll(m & below_mask);
        const uint32_t c0 = valid ? wc[d] : 0u;
        if (valid && below == 0) wc[d] = (uint16_t)(c0 + (uint32_t)__popcll(m));
        dig[r] = d | (c0 + below) << 16;
    }
    __syncthreads();
    // tile positions: exclusive sums over the digits (`per` consecutive ones a thread), then over the waves
    const int per = (D + THREADS - 1) / THREADS;
    uint32_t s = 0;
    for (int q = 0; q < per; q++) {
        const int d = tid * per + q;
        if (d < D)
            for (int v = 0; v < WAVES; v++) s += wcnt[v * D + d];
    }
    uint32_t incl = s;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    uint32_t run = incl - s;
    for (int v = 0; v < w; v++) run += wsum[v];
    for (int q = 0; q < per; q++) {
        const int d = tid * per + q;
        if (d < D) {
            const uint32_t first = OUT == kSegPart ? a.rows[(int64_t)d * gridDim.x + blockIdx.x]
                                                   : a.rows[(int64_t)blockIdx.x * D + d] + a.dbase[(int64_t)run_of * D + d];
            gd[d] = first - run;
            for (int v = 0; v < WAVES; v++) {
                const uint32_t c = wcnt[v * D + d];
                wcnt[v * D + d] = (uint16_t)run;
                run += c;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; r++) {
        dig[r] = span + r * 64 < un ? wc[dig[r] & 0xffffu] + (dig[r] >> 16) : 0xffffffffu;
    }
    for (int c0 = 0; c0 < count; c0 += STAGE) {
#pragma unroll
        for (int r = 0; r < ITEMS; r++) {
            const uint32_t q = dig[r] - (uint32_t)c0;
            if (q < (uint32_t)STAGE) {
                const uint32_t i = span + r * 64;
                const int32_t from = kFromPos ? (int32_t)base + (int32_t)i : ei[kFromPos ? 0 : r];
                stage[q] = make_float4(ex[r], ey[r], ez[r], __int_as_float(from));
                skey[q] = kin[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < STAGE / THREADS; r++) {
            const int q = r * THREADS + tid;
            if (c0 + q < count) {
                const int32_t k = skey[q];
                const float4 v = stage[q];
                const uint32_t dest = gd[((uint32_t)k >> a.shift) & mask] + (uint32_t)(c0 + q);
                a.kout[dest] = k;
                if constexpr (OUT == kSegPart || OUT == kSegMid) {
                    a.out[dest] = v;
                } else {
                    const int b = a.n_boxes > 1 ? box_of_cell(a.boxes, a.n_boxes, k) : 0;
                    a.out[dest] = cell_relative(v.x, v.y, v.z, a.boxes[b]);
                    a.vout[dest] = __float_as_int(v.w);
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------- cell offsets and layout

__global__ void k_run_ends(const int32_t *__restrict__ keys, int64_t n, int32_t *__restrict__ endpos) {
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n) return;
    int32_t k = keys[s];
    if (s == n - 1 || keys[s + 1] != k) endpos[k] = (int32_t)(s + 1);
}

}  // namespace

// ---------------------------------------------------------------- host launchers

hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n, 256)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_set_boxes(const abacus_nf_box *boxes, int n_boxes, const int32_t *cell_base, BoxDev *dst,
                            hipStream_t st) {
    for (int first = 0; first < n_boxes; first += kBoxChunk) {
        BoxChunk c;
        memset(&c, 0, sizeof(c));
        c.first = first;
        c.count = n_boxes - first < kBoxChunk ? n_boxes - first : kBoxChunk;
        for (int k = 0; k < c.count; k++) {
            const abacus_nf_box &b = boxes[first + k];
            c.b[k].offset = b.offset;
            c.b[k].n = b.n;
            c.b[k].L = b.box;
            c.b[k].s = (double)b.K / b.box;
            c.b[k].K = b.K;
            c.b[k].cell_base = cell_base[first + k];
        }
        hipLaunchKernelGGL(k_set_boxes, dim3(1), dim3(kBoxChunk), 0, st, c, dst);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

size_t scan_temp_bytes(int64_t n) { return scan_levels_bytes(n, sizeof(int64_t)) + 1024; }

hipError_t scan_i32_max_inclusive(const int32_t *in, int32_t *out, int64_t n, void *temp, hipStream_t st) {
    return scan_impl<int32_t, OpMax>(in, out, n, true, (int32_t)0, (char *)temp, st);
}

namespace {

template <int THREADS, int ITEMS, int OUT>
hipError_t scatter(const SegArgs &a, unsigned grid, hipStream_t st) {
    const size_t D = (size_t)1 << a.bits;
    const size_t stage = std::min(THREADS * ITEMS, kStageMost);
    const size_t lds = 20 * stage + 4 * D + 4 * (THREADS / 64) + 2 * (THREADS / 64) * D;
    auto k = k_seg_scatter<THREADS, ITEMS, OUT>;
    if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3(grid), dim3(THREADS), lds, st, a);
    return hipGetLastError();
}

template <int THREADS, int ITEMS>
hipError_t sort_impl(const SortArgs &a, const SortPlan &pl, int bits, int32_t **keys_out, bool *have_starts,
                     hipStream_t st) {
    constexpr int TILE = THREADS * ITEMS;
    const int64_t n = a.n;
    const int ntiles = (int)((n + TILE - 1) / TILE);
    const SortScratch at = sort_scratch(n, pl);
    Buckets *bk = (Buckets *)a.temp;
    uint32_t *dbase = (uint32_t *)((char *)a.temp + at.dbase), *rows = (uint32_t *)((char *)a.temp + at.rows);
    const int first = pl.part ? pl.part : pl.last;
    hipLaunchKernelGGL((k_bin<THREADS, ITEMS>), dim3(ntiles), dim3(THREADS), sizeof(uint32_t) << first, st, a.pos, n,
                       a.boxes, a.n_boxes, a.keys_a, pl.part ? bits - pl.part : 0, first, rows, pl.part ? 0 : 1, a.err);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    SegArgs s;
    s.kin = a.keys_a;
    s.pos = a.pos;
    s.pay = a.pay;
    s.rows = rows;
    s.dbase = dbase;
    s.bk = nullptr;
    s.nb = 1 << pl.part;
    s.boxes = a.boxes;
    s.n_boxes = a.n_boxes;
    s.n = n;
    s.shift = 0;
    s.bits = pl.last;
    s.run_shift = run_shift(n);
    s.vout = a.perm;
    s.out = a.spos;
    *have_starts = pl.mid == 0;
    const int nb = 1 << pl.part, shift_runs = s.run_shift;
    // first slots of a digit of nbits bits from the tiles' counts
    auto sums = [&](Buckets *buckets, int nbits, bool starts) {
        const int runs = buckets ? (ntiles >> shift_runs) + nb : (int)((ntiles + ((int64_t)1 << shift_runs) - 1) >> shift_runs);
        const bool single = ntiles <= (1 << shift_runs);
        int32_t *cell_start = starts ? a.cell_start : nullptr;
        hipLaunchKernelGGL(k_seg_sums, dim3(runs), dim3(kSegScanThreads), 0, st, rows, dbase, buckets, nb, n, ntiles,
                           shift_runs, nbits, (int)single, cell_start, a.n_cells);
        hipError_t r = hipGetLastError();
        if (r != hipSuccess || single || buckets) return r;
        hipLaunchKernelGGL(k_seg_base, dim3(1), dim3(kSegScanThreads), 0, st, dbase, n, runs, nbits, cell_start, a.n_cells);
        return hipGetLastError();
    };
    if (!pl.part) {
        if ((e = sums(nullptr, pl.last, true)) != hipSuccess) return e;
        s.kout = *keys_out = a.keys_b;
        return scatter<THREADS, ITEMS, kSegLastPos>(s, ntiles, st);
    }
    uint32_t *toff = rows + (size_t)nb * ntiles;
    char *scan_tmp = (char *)(((uintptr_t)(toff + (size_t)nb * ntiles) + 255) & ~(uintptr_t)255);
    e = scan_impl<uint32_t, OpAdd>(rows, toff, (int64_t)nb * ntiles, false, 0u, scan_tmp, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_buckets, dim3(1), dim3(kMaxBuckets), 0, st, toff, ntiles, nb, n, TILE, shift_runs, bk);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    SegArgs q = s;
    q.rows = toff;
    q.shift = bits - pl.part;
    q.bits = pl.part;
    q.kout = a.keys_b;
    q.vout = nullptr;
    q.out = pl.mid ? a.spos : a.pay;   // the coordinates end up in pay before the last scatter
    if ((e = scatter<THREADS, ITEMS, kSegPart>(q, ntiles, st)) != hipSuccess) return e;
    s.bk = bk;
    const unsigned grid = (unsigned)(ntiles + nb);   // at least the tiles of all buckets
    auto digit = [&](const int32_t *keys, int shift, int nbits, bool starts) {
        hipLaunchKernelGGL((k_seg_hist<THREADS, ITEMS>), dim3(grid), dim3(THREADS), sizeof(uint32_t) << nbits, st, keys,
                           n, bk, nb, shift, nbits, rows);
        hipError_t r = hipGetLastError();
        if (r != hipSuccess) return r;
        return sums(bk, nbits, starts);
    };
    if (!pl.mid) {
        s.kin = a.keys_b;
        s.kout = *keys_out = a.keys_a;
        if ((e = digit(a.keys_b, 0, pl.last, true)) != hipSuccess) return e;
        return scatter<THREADS, ITEMS, kSegLast>(s, grid, st);
    }
    if ((e = digit(a.keys_b, 0, pl.mid, false)) != hipSuccess) return e;
    SegArgs m = s;
    m.kin = a.keys_b;
    m.pay = a.spos;
    m.bits = pl.mid;
    m.kout = a.keys_a;
    m.out = a.pay;
    if ((e = scatter<THREADS, ITEMS, kSegMid>(m, grid, st)) != hipSuccess) return e;
    if ((e = digit(a.keys_a, pl.mid, pl.last, false)) != hipSuccess) return e;
    s.kin = a.keys_a;
    s.shift = pl.mid;
    s.kout = *keys_out = a.keys_b;
    return scatter<THREADS, ITEMS, kSegLast>(s, grid, st);
}

}  // namespace

hipError_t sort_by_cell(const SortArgs &a, int key_bits, int32_t **keys_out, bool *have_starts, hipStream_t st) {
    *keys_out = a.keys_a;
    *have_starts = false;
    if (a.n <= 0) return hipSuccess;
    const SortPlan pl = sort_plan(a.n, key_bits);
    switch (tile_class(a.n)) {
        case 0: return sort_impl<256, 4>(a, pl, key_bits, keys_out, have_starts, st);
        case 1: return sort_impl<256, 8>(a, pl, key_bits, keys_out, have_starts, st);
        default: return sort_impl<kBigThreads, kBigItems>(a, pl, key_bits, keys_out, have_starts, st);
    }
}

hipError_t launch_cell_start(const int32_t *keys_sorted, int64_t n, int64_t n_cells, int32_t *endpos,
                             int32_t *cell_start, void *scan_temp, hipStream_t st) {
    hipError_t e = launch_fill_i32(endpos, n_cells, 0, st);
    if (e != hipSuccess) return e;
    e = launch_fill_i32(cell_start, 1, 0, st);
    if (e != hipSuccess) return e;
    if (n > 0) {
        hipLaunchKernelGGL(k_run_ends, dim3(grid_for(n, 256)), dim3(256), 0, st, keys_sorted, n, endpos);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return scan_i32_max_inclusive(endpos, cell_start + 1, n_cells, scan_temp, st);
}

}  // namespace anf
