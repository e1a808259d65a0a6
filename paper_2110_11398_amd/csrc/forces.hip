// Near-field force: device work list and the persistent pairwise kernel.
//
// The operation is the direct sum of Sec. 3.1 (near field = cells within R,
// explicit periodic images) with the spline or Plummer softening of Sec. 2.5
// and Sec. 5.2.  The paper runs it as CUDA kernels on host-packaged work units
// ("Index Near Force Pencils", "spatially compact GPU work units", Sec. 4.3 and
// Sec. 4.5).  Here the work list is built on the device and one persistent
// launch drains it:
//
//   k_wl_cells    per cell: occupancy n_c, near-field source count; per box: pair and work totals
//   k_wl_plan     the source-part length of every box, and up to which length a cell is not split over items
//   k_wl_bins,    where the lists are short: what splitting the cells of every length takes, and which stay whole
//   k_wl_fit      so that the rest fits
//   k_wl_count    per cell: items, partial slots, cost class (histogram over classes)
//   k_wl_emit     class offsets (heaviest items first), capacity checks, items in class order
//   k_forces      persistent waves pop items: sink tile in VGPRs, sources staged
//                 through the wave's LDS region with the periodic cell offset
//                 applied, FP32 pair math, FP32 / two-sum / FP64 accumulation,
//                 ordered cross-lane reduction, output in input order
//   k_finalize    sums the parts of sinks whose source list was split (FP64)
//
// Numbers are in cell-width units: positions are relative to the sink cell's
// centre, so the pair terms need no large-coordinate cancellation.
#include <algorithm>
#include <climits>
#include <cstring>
#include <cmath>

#include "nf_internal.h"

namespace anf {

namespace {

constexpr int kWaves = 4;                 // independent waves per workgroup
constexpr int kThreads = 64 * kWaves;
constexpr int kRounds = 4;                // source slots per lane of a staged chunk
constexpr int kMaxCols = 49;              // near-field columns at the largest R
constexpr int kGroupPairs = 8;            // pairs of a lane whose reciprocal square roots go together
constexpr float kTiny = 1e-20f;           // keeps rsqrt finite for coincident pairs
constexpr float kFar = 1e18f;             // padding source: its terms underflow to exactly 0

inline unsigned grid_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

// ---------------------------------------------------------------- per-box constants

constexpr int kFBoxChunk = 48;
struct FBoxChunk {
    ForceBox f[kFBoxChunk];
    int first, count;
};

// Clears the work state and the totals of boxes [first, first + count) for a new work list.
__device__ inline void clear_work(WorkState *ws, WorkBox *wb, int first, int count, int grid) {
    const int t = threadIdx.x;
    for (int i = t; i < count; i += blockDim.x) wb[first + i] = WorkBox{0, 0, 0, 0, 0, 0};
    if (first != 0) return;
    if (t == 0) {
        ws->partial_slots = 0;
        ws->n_items = 0;
        ws->overflow = 0;
        ws->pairs = 0;
        ws->whole_bin = -1;
        ws->whole_slots = ws->whole_items = 0;
    }
    // the first slots of every queue belong to the waves that start on it
    if (t < kQueues) ws->cursor[t][0] = grid > t ? (grid - t + kQueues - 1) / kQueues * kWaves : 0;
    if (t < kNumClasses) {
        ws->class_count[t] = 0;
        ws->class_fill[t] = 0;
        ws->bin_slots[t] = 0;
        ws->bin_items[t] = 0;
    }
}

__global__ __launch_bounds__(64) void k_set_fbox(FBoxChunk c, ForceBox *dst, WorkState *ws, WorkBox *wb, int grid) {
    static_assert(kNumClasses <= 64 && kFBoxChunk <= 64, "one lane each");
    const int i = threadIdx.x;
    if (i < c.count) dst[c.first + i] = c.f[i];
    clear_work(ws, wb, c.first, c.count, grid);
}

__global__ __launch_bounds__(64) void k_wl_clear(WorkState *ws, WorkBox *wb, int n_boxes) {
    clear_work(ws, wb, 0, n_boxes, 0);
}

// ---------------------------------------------------------------- near-field columns

// The near field of cell (cx, cy, cz) is (2R+1)^2 columns of neighbouring
// cells, each a run of 2R+1 consecutive cells along z.  In the sorted layout
// a run is a contiguous slot range, split in two where it wraps through the
// periodic z boundary.  czref turns the stored z cell index of a source into
// its offset from the sink cell: dz = cz_src - czref.
struct ColSeg {
    int32_t src0, len0, src1, len1;
    float czref0, czref1;
};

__device__ inline void column_segments(const int32_t *__restrict__ cs, int colbase, int cz, int K, int R,
                                       ColSeg &o) {
    const int z0 = cz - R, z1 = cz + R;
    if (z0 < 0) {            // images below the box first, then the cells from 0
        o.src0 = cs[colbase + z0 + K];
        o.len0 = cs[colbase + K] - o.src0;
        o.czref0 = (float)(cz + K);
        o.src1 = cs[colbase];
        o.len1 = cs[colbase + z1 + 1] - o.src1;
        o.czref1 = (float)cz;
    } else if (z1 >= K) {    // cells up to K-1, then images above the box
        o.src0 = cs[colbase + z0];
        o.len0 = cs[colbase + K] - o.src0;
        o.czref0 = (float)cz;
        o.src1 = cs[colbase];
        o.len1 = cs[colbase + z1 - K + 1] - o.src1;
        o.czref1 = (float)(cz - K);
    } else {
        o.src0 = cs[colbase + z0];
        o.len0 = cs[colbase + z1 + 1] - o.src0;
        o.czref0 = (float)cz;
        o.src1 = 0;
        o.len1 = 0;
        o.czref1 = 0.f;
    }
}

__device__ inline int wrap(int v, int K) { return v < 0 ? v + K : (v >= K ? v - K : v); }

// Number of near-field sources of a cell: the loads of all columns in flight at once.
template <int R>
__device__ inline int cell_sources(const int32_t *__restrict__ cs, const BoxDev &B, int lin) {
    const int K = B.K;
    const int cz = lin % K, cy = (lin / K) % K, cx = lin / (K * K);
    int total = 0;
#pragma unroll
    for (int dx = -R; dx <= R; dx++) {
        const int ex = wrap(cx + dx, K);
#pragma unroll
        for (int dy = -R; dy <= R; dy++) {
            const int ey = wrap(cy + dy, K);
            ColSeg o;
            column_segments(cs, B.cell_base + (ex * K + ey) * K, cz, K, R, o);
            total += o.len0 + o.len1;
        }
    }
    return total;
}

// Source iterations per lane of a cell's first tile (fewest lanes per group).
__device__ inline int cell_iters(int n, int nsrc, int S, int max_lanes) {
    const int L0 = tile_at(n, S, max_lanes, 0).L;
    return (nsrc + L0 - 1) / L0;
}

// Cost class of a cell's items: one part of its source list against its first tile, iterations per lane x sinks
// per lane; classes are half octaves, heaviest first.  The tiles of a cell's rest are lighter and share the
// class on purpose: they wait on their loads more than they compute, and run best among heavier items (with a
// class of their own, at the end of the list: uniform box of 2097152 particles 4.77 -> 5.07 ms).
__device__ inline int cell_class(int iters, int S, int parts) {
    const float cost = (float)(iters / parts + 1) * (float)S + 16.0f;
    const int cls = kNumClasses - 1 - (int)(2.0f * log2f(cost));
    return cls < 0 ? 0 : (cls >= kNumClasses ? kNumClasses - 1 : cls);
}

// ---------------------------------------------------------------- work-list kernels

__device__ inline unsigned long long wave_sum_u64(unsigned long long v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Per cell: source count; per box: exact pair total, unsplit items, and the sums that bound the partial slots
// and items of a part length (slots <= n + slot_iters / length, items <= tiles + item_iters / length).  Also
// clears the per-cell maxima of |a|^2 the force pass is about to record.  Additions to one box's totals take
// turns on their cache line and are kept few: with one box, workgroups walk the cells in strides and add once
// (one addition per wave: 0.81 ms in a late-time box of 4.2 million cells); in a batch, every wave walks a run
// of consecutive cells and adds when the box changes (strides, with each thread adding at every box it met,
// took 25.8 ms for 64 boxes of 3.4 million cells in all; this takes 0.67 with the rest of the list).
template <int R>
__global__ __launch_bounds__(256) void k_wl_cells(const int32_t *__restrict__ cs, const BoxDev *__restrict__ boxes,
                                                  int n_boxes, int64_t n_cells, int S, int max_lanes,
                                                  int32_t *__restrict__ cell_nsrc,
                                                  unsigned long long *__restrict__ amax, WorkBox *__restrict__ wb) {
    __shared__ unsigned long long part[4][4];
    unsigned long long v[4] = {0, 0, 0, 0};   // pairs, slot_iters, item_iters, tiles of the open box
    // adds one cell's share to w and records its source count
    auto count = [&](int64_t c, int n, int b, unsigned long long *w) {
        int nsrc = 0;
        if (n > 0) {
            const BoxDev B = boxes[b];
            nsrc = cell_sources<R>(cs, B, (int)(c - B.cell_base));
            const int tiles = tile_count(n, S, max_lanes);
            const unsigned long long iters = (unsigned long long)cell_iters(n, nsrc, S, max_lanes);
            w[0] += (unsigned long long)n * (unsigned long long)nsrc;
            w[1] += (unsigned long long)n * iters;
            w[2] += (unsigned long long)tiles * iters;
            w[3] += (unsigned long long)tiles;
        }
        cell_nsrc[c] = nsrc;
        if (amax) amax[c] = 0;
    };
    if (n_boxes > 1) {
        const int lane = threadIdx.x & 63;
        const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), waves = (int64_t)gridDim.x * 4;
        const int64_t run = (n_cells + waves * 64 - 1) / (waves * 64) * 64;
        const int64_t first = wave * run, end = first + run < n_cells ? first + run : n_cells;
        int open = -1;
        auto flush = [&]() {   // the whole wave
            if (open < 0) return;
#pragma unroll
            for (int q = 0; q < 4; q++) v[q] = wave_sum_u64(v[q]);
            if (lane == 0) {
                atomicAdd(&wb[open].pairs, v[0]);
                atomicAdd(&wb[open].slot_iters, v[1]);
                atomicAdd(&wb[open].item_iters, v[2]);
                atomicAdd(&wb[open].tiles, v[3]);
            }
            v[0] = v[1] = v[2] = v[3] = 0;
        };
        for (int64_t c0 = first; c0 < end; c0 += 64) {
            const int64_t c = c0 + lane;
            unsigned long long w[4] = {0, 0, 0, 0};
            int b = -1;   // stays so for an empty cell, which adds nothing
            if (c < end) {
                const int n = cs[c + 1] - cs[c];
                if (n > 0) b = box_of_cell(boxes, n_boxes, (int32_t)c);
                count(c, n, b, w);
            }
            for (unsigned long long left = __ballot(b >= 0); left;) {
                const int x = __builtin_amdgcn_readlane(b, __ffsll((long long)left) - 1);
                if (x != open) {
                    flush();
                    open = x;
                }
                if (b == x)
#pragma unroll
                    for (int q = 0; q < 4; q++) v[q] += w[q];
                left &= ~__ballot(b == x);
            }
        }
        flush();
        return;
    }
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < n_cells; c += (int64_t)gridDim.x * blockDim.x)
        count(c, cs[c + 1] - cs[c], 0, v);
#pragma unroll
    for (int q = 0; q < 4; q++) {
        v[q] = wave_sum_u64(v[q]);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][q] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        const int q = threadIdx.x;
        const unsigned long long t = part[0][q] + part[1][q] + part[2][q] + part[3][q];
        if (t) atomicAdd((q == 0 ? &wb[0].pairs : q == 1 ? &wb[0].slot_iters : q == 2 ? &wb[0].item_iters : &wb[0].tiles), t);
    }
}

// Source iterations per lane of a wave's share of `pairs` pairs, at most part_sources.
__device__ inline int fill_length(unsigned long long pairs, int S, int part_sources) {
    const unsigned long long fill = (pairs / (64 * kFillItems)) >> (S >> 1);   // S is 1, 2 or 4
    return fill > (unsigned long long)part_sources ? part_sources : (int)fill;
}

// Length of the source parts of every box (source iterations per lane).  A box is cut so that its work gives
// at least about kFillItems equal items: an item of a heavy cell that is longer than a wave's share of the box
// leaves the rest of the chip idle until it ends.  The length is at most the tuning's part_sources and at least
// kMinPart (twice that where such parts still give kFewItems items), and longer where the box's own room (box_slots,
// box_items) is less than its parts would take: it follows from the box alone, so a box gives bit-identical forces
// whatever batch it is in.
//
// What a batch decides is which cells are split over items at all.  A cell whose list is no longer than a wave's share
// of the whole batch stays one item per tile, which goes through the parts in order and adds them up as k_finalize
// would: no slots to write and read again (512 boxes of 32768 uniform particles: 41.6 ms with every cell split over
// items, 40.8 with whole ones, the same bits).
__global__ __launch_bounds__(256) void k_wl_plan(WorkState *__restrict__ ws, WorkBox *__restrict__ wb,
                                                 const BoxDev *__restrict__ boxes, int n_boxes, int S,
                                                 int part_sources) {
    __shared__ unsigned long long pairs;   // of this workgroup's boxes
    if (threadIdx.x == 0) pairs = 0;
    __syncthreads();
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b < n_boxes) {
        const WorkBox w = wb[b];
        const int64_t n = boxes[b].n, K = boxes[b].K;
        const long long want = fill_length(w.pairs, S, part_sources), least = least_part(w.pairs, S);
        const long long it = want < least ? least : want;
        // bounds at this length: slots <= n + slot_iters / length, items <= tiles + item_iters / length
        const double slots = (double)w.slot_iters / (double)it + 1.0, items = (double)w.item_iters / (double)it + 1.0;
        const double slot_room = (double)(box_slots(n) - n), item_room = (double)box_items(n, K * K * K) - (double)w.tiles;
        double f = 1.0;
        if (slots > slot_room) f = slot_room >= 1.0 ? slots / slot_room : 1e18;
        if (items > item_room) f = fmax(f, item_room >= 1.0 ? items / item_room : 1e18);
        const double v = f > 1.0 ? ceil((double)it * (f * (1.0 + 1e-9))) : (double)it;
        wb[b].part_iters = v > (double)INT_MAX ? INT_MAX : (int32_t)v;
        if (w.pairs) atomicAdd(&pairs, w.pairs);
    }
    __syncthreads();
    if (threadIdx.x == 0 && pairs) atomicAdd(&ws->pairs, pairs);
}

// Length bin of a cell's source list: half octaves of its source iterations.
__device__ inline int length_bin(int iters) {
    const int b = (int)(2.0f * log2f((float)iters));
    return b < 0 ? 0 : (b >= kNumClasses ? kNumClasses - 1 : b);
}

// Parts of the source list of a cell that is not empty: as many as keep its first tile at about part_iters source
// iterations per lane; negative where they stay together in one item per tile.
__device__ inline int cell_split(int iters, int nsrc, int part_iters, int whole_iters, int whole_bin) {
    int parts = (int)(((unsigned)iters + (unsigned)part_iters - 1u) / (unsigned)part_iters);
    if (parts > nsrc) parts = nsrc;
    if (parts <= 1) return 1;
    return iters <= whole_iters || (whole_bin >= 0 && length_bin(iters) <= whole_bin) ? -parts : parts;
}

// Where the boxes' rooms add up to more than the lists hold: what splitting the cells of every length bin takes.
__global__ __launch_bounds__(256) void k_wl_bins(const int32_t *__restrict__ cs, const int32_t *__restrict__ cell_nsrc,
                                                 const BoxDev *__restrict__ boxes, int n_boxes, int64_t n_cells, int S,
                                                 int max_lanes, int part_sources, const WorkBox *__restrict__ wb,
                                                 WorkState *ws) {
    const int whole_iters = fill_length(ws->pairs, S, part_sources);
    __shared__ unsigned long long slots[kNumClasses + 1], items[kNumClasses + 1];   // the last: with every cell whole
    if (threadIdx.x <= kNumClasses) slots[threadIdx.x] = items[threadIdx.x] = 0;
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int n = c < n_cells ? cs[c + 1] - cs[c] : 0;
    if (n > 0) {
        const int b = n_boxes > 1 ? box_of_cell(boxes, n_boxes, (int32_t)c) : 0;
        const int nsrc = cell_nsrc[c], iters = cell_iters(n, nsrc, S, max_lanes);
        const int parts = cell_split(iters, nsrc, wb[b].part_iters, whole_iters, -1);
        const unsigned long long tiles = (unsigned long long)tile_count(n, S, max_lanes);
        atomicAdd(&items[kNumClasses], tiles);
        if (parts < 0 || parts > 1) atomicAdd(&slots[kNumClasses], (unsigned long long)n);
        if (parts > 1) {
            const int bin = length_bin(iters);
            atomicAdd(&slots[bin], (unsigned long long)n * (unsigned long long)(parts - 1));
            atomicAdd(&items[bin], tiles * (unsigned long long)(parts - 1));
        }
    }
    __syncthreads();
    if (threadIdx.x <= kNumClasses) {
        const int k = threadIdx.x;
        if (slots[k]) atomicAdd(k < kNumClasses ? &ws->bin_slots[k] : &ws->whole_slots, slots[k]);
        if (items[k]) atomicAdd(k < kNumClasses ? &ws->bin_items[k] : &ws->whole_items, items[k]);
    }
}

// The shortest lists stay whole, bin by bin, until the others fit: one lane per bin.
__global__ __launch_bounds__(64) void k_wl_fit(WorkState *ws, int64_t partial_capacity, int64_t item_capacity) {
    static_assert(kNumClasses == 64, "one lane per bin");
    const int k = threadIdx.x;
    unsigned long long slots = ws->bin_slots[k], items = ws->bin_items[k];   // then of bins k and up
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long s = __shfl_down(slots, off), i = __shfl_down(items, off);
        if (k + off < 64) {
            slots += s;
            items += i;
        }
    }
    const unsigned long long too_many = __ballot(ws->whole_slots + slots > (unsigned long long)partial_capacity ||
                                                 ws->whole_items + items > (unsigned long long)item_capacity);
    if (k == 0) ws->whole_bin = 63 - __clzll((long long)too_many);   // -1: all fit
}

__global__ __launch_bounds__(256) void k_wl_count(const int32_t *__restrict__ cs, const int32_t *__restrict__ cell_nsrc,
                                                  const BoxDev *__restrict__ boxes, int n_boxes, int64_t n_cells, int S,
                                                  int max_lanes, int part_sources, const WorkBox *__restrict__ wb,
                                                  WorkState *ws, int32_t *__restrict__ cell_parts,
                                                  int64_t *__restrict__ cell_pbase) {
    const int whole_iters = fill_length(ws->pairs, S, part_sources);
    __shared__ int32_t hist[kNumClasses];
    __shared__ unsigned long long need, base;   // partial slots of this workgroup's split cells
    if (threadIdx.x < kNumClasses) hist[threadIdx.x] = 0;
    if (threadIdx.x == 0) need = 0;
    __syncthreads();
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long local = 0;
    int parts = 0;
    if (c < n_cells) {
        const int n = cs[c + 1] - cs[c], nsrc = cell_nsrc[c];
        if (n > 0) {
            const int b = n_boxes > 1 ? box_of_cell(boxes, n_boxes, (int32_t)c) : 0;
            const int iters = cell_iters(n, nsrc, S, max_lanes);
            parts = cell_split(iters, nsrc, wb[b].part_iters, whole_iters, ws->whole_bin);
            const int split = parts < 0 ? 1 : parts;
            if (parts != 1) local = atomicAdd(&need, (unsigned long long)split * (unsigned long long)n);
            atomicAdd(&hist[cell_class(iters, S, split)], tile_count(n, S, max_lanes) * split);
        }
        cell_parts[c] = parts;
    }
    __syncthreads();
    if (threadIdx.x == 0) base = need ? atomicAdd(&ws->partial_slots, need) : 0;
    if (threadIdx.x < kNumClasses && hist[threadIdx.x]) atomicAdd(&ws->class_count[threadIdx.x], hist[threadIdx.x]);
    __syncthreads();
    if (parts < 0 || parts > 1) cell_pbase[c] = (int64_t)(base + local);
}

// Items in class order.  Every workgroup forms the class offsets (heaviest class first) from the counts; the
// first one also records the item count, the capacity check and where the light items start in each queue.
__global__ __launch_bounds__(256) void k_wl_emit(const int32_t *__restrict__ cs, const int32_t *__restrict__ cell_nsrc,
                                                 const int32_t *__restrict__ cell_parts,
                                                 const BoxDev *__restrict__ boxes, int n_boxes, int64_t n_cells,
                                                 int S, int max_lanes, WorkState *ws,
                                                 Item *__restrict__ items, int64_t item_capacity,
                                                 int64_t partial_capacity, int per_block, int *err) {
    __shared__ int32_t cnt[kNumClasses];
    __shared__ int64_t cbase[kNumClasses];
    __shared__ int32_t over;
    __shared__ int32_t end[256], ntile[256], cbox[256], wsum[4];
    __shared__ int64_t first[256];
    static_assert(kNumClasses == 64, "one lane per class");
    if (threadIdx.x < kNumClasses) {
        const int k = threadIdx.x;
        cnt[k] = 0;
        const int64_t own = ws->class_count[k];
        int64_t incl = own;
        for (int off = 1; off < 64; off <<= 1) {
            const int64_t y = __shfl_up(incl, off);
            if (k >= off) incl += y;
        }
        cbase[k] = incl - own;
        const int64_t run = __shfl(incl, 63);
        // on overflow nothing is emitted and nothing is computed: the error is
        // reported by abacus_nf_sync and the output is left unwritten
        const int o = run > item_capacity || (int64_t)ws->partial_slots > partial_capacity ? 1 : 0;
        const int64_t L0 = __shfl(incl - own, kLightClass);
        if (k == 0) over = o;
        if (blockIdx.x == 0) {
            if (k == 0) {
                ws->n_items = o ? 0 : (int32_t)run;
                ws->overflow = o;
                if (o) atomicCAS(err, 0, ABACUS_NF_ECAPACITY);
            }
            // slot j of queue x holds item ((j / kQueueBlock) * kQueues + x) * kQueueBlock + j % kQueueBlock,
            // increasing in j: the first slot of each queue at or past the first light item
            const int64_t B = L0 / kQueueBlock, r = L0 % kQueueBlock;
            if (k < kQueues) {
                const int64_t bq = B > k ? (B - k + kQueues - 1) / kQueues : 0;   // first block of queue k at or past B
                const int64_t slot = bq * kQueueBlock + (bq * kQueues + k == B ? r : 0);
                ws->light_slot[k] = (int32_t)(slot < INT_MAX ? slot : INT_MAX);
            }
        }
    }
    __syncthreads();
    const int64_t c0 = (int64_t)blockIdx.x * per_block, c = c0 + threadIdx.x;
    int tiles = 0, parts = 0, cls = 0, local = 0, b = 0;
    if ((int)threadIdx.x < per_block && c < n_cells && !over) {
        const int n = cs[c + 1] - cs[c];
        if (n > 0) {
            b = n_boxes > 1 ? box_of_cell(boxes, n_boxes, (int32_t)c) : 0;
            parts = cell_parts[c] < 0 ? 1 : cell_parts[c];
            tiles = tile_count(n, S, max_lanes);
            cls = cell_class(cell_iters(n, cell_nsrc[c], S, max_lanes), S, parts);
            local = atomicAdd(&cnt[cls], tiles * parts);
        }
    }
    __syncthreads();
    if (threadIdx.x < kNumClasses) {
        const int k = threadIdx.x;
        if (cnt[k]) cbase[k] += atomicAdd(&ws->class_fill[k], cnt[k]);
    }
    __syncthreads();
    // The items of the workgroup's cells are written by all of its threads (a halo core alone has thousands),
    // part-major within a cell: consecutive items are the tiles of one source part, so the waves that take them
    // together (one queue block goes to one XCD) stream the same sources through that XCD's L2.
    const int own = tiles * parts;
    int incl = own;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off);
        if ((int)(threadIdx.x & 63) >= off) incl += y;
    }
    if ((threadIdx.x & 63) == 63) wsum[threadIdx.x >> 6] = incl;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < (int)(threadIdx.x >> 6); w++) before += wsum[w];
    end[threadIdx.x] = before + incl;
    first[threadIdx.x] = cbase[cls] + local;
    ntile[threadIdx.x] = tiles;
    cbox[threadIdx.x] = b;
    __syncthreads();
    const int total = end[255];
    for (int i = threadIdx.x; i < total; i += 256) {
        int lo = 0, hi = 255;   // the first cell whose items end past i
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (end[mid] > i) hi = mid; else lo = mid + 1;
        }
        const int j = i - (lo > 0 ? end[lo - 1] : 0), nt = ntile[lo];
        const int64_t k = first[lo] + j;
        if (k < item_capacity) items[k] = Item{(int32_t)(c0 + lo), j % nt, j / nt, cbox[lo]};
    }
}

// ---------------------------------------------------------------- the force kernel

struct KArgs {
    const float4 *spos;
    const int32_t *cs;
    const int32_t *perm;
    const Item *items;
    WorkState *ws;
    const BoxDev *boxes;
    const ForceBox *fbox;
    const int32_t *cell_parts;
    const int64_t *cell_pbase;
    double *partials;
    float *acc;
    double *acc64;  // FP64 accelerations instead of acc when not null
    float *rho;
    unsigned long long *amax;   // [n_cells] bits of the largest |a|^2 written in each cell
    int R;
    int chunk;      // sources per LDS chunk (at most 64 * kRounds)
    int max_lanes;
    int region;     // bytes of LDS per wave
};

// Offsets of the sources of one near-field column, in LDS: entry 2 c + i for run i of column c.
struct ColOff {
    float x, y, czref;
};

// Second run of a column that wraps through the box boundary: its first slot in the flattened list, and what to add
// to a flattened slot there to get the slot of the source.
struct ColWrap {
    int32_t split, base;
};

constexpr size_t kColBytes = 2 * kMaxCols * sizeof(ColOff) + kMaxCols * sizeof(ColWrap);

// Orders LDS traffic between the lanes of one wave (no other wave takes part).
__device__ inline void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ inline int sgpr(int v) { return __builtin_amdgcn_readfirstlane(v); }

// A wave-uniform float held in a scalar register.
__device__ inline float uniform(float v) { return __builtin_bit_cast(float, sgpr(__builtin_bit_cast(int, v))); }

// Knuth's two-sum: s + e == a + b exactly.
__device__ __forceinline__ void two_sum(float a, float b, float &s, float &e) {
    s = a + b;
    const float bp = s - a;
    e = (a - (s - bp)) + (b - bp);
}

// |a|^2 of a written acceleration: FP64 squares of the stored values, each rounded, summed in a fixed order.
__device__ inline double norm2_written(double x, double y, double z) {
#pragma clang fp contract(off)
    return x * x + y * y + z * z;
}

// Largest |a|^2 of a cell: the bit patterns of non-negative doubles order like their values, so an
// integer maximum is exact and independent of the order of the updates.
__device__ inline void cell_max(unsigned long long *amax, int c, double v) {
    atomicMax(amax + c, (unsigned long long)__double_as_longlong(v));
}

__device__ inline double wave_max_f64(double v) {
    for (int off = 32; off > 0; off >>= 1) {
        const double y = __shfl_xor(v, off);
        v = v > y ? v : y;
    }
    return v;
}

// U staged sources against the S sinks of this lane.  With KDE, also the
// density weight max(0, 1 - r^2/b^2) = max(0, kc - r2 * ib2) (r2 carries the
// pair chain's constant offset, folded into kc).
//
// The loop is bound by VALU issue.  A SIMD issues the plain FP32 operations of two waves at a time (2 clocks a
// wave instruction), the reciprocal square root alone (8 clocks), so the 12 operations of a pair cost 30 clocks
// when the waves stay paired.  They do not by themselves: a wave that comes out of its reciprocal square roots
// while the others wait for theirs runs alone for a while (measured on a loop of these 12 operations: 48 clocks a
// pair at six waves per SIMD).  So the reciprocal square roots of up to kGroupPairs pairs are issued together at
// raised wave priority: once one wave has started, the others reach theirs before plain work goes on, and all
// come out in step (33 clocks a pair in the same loop).  Clustered box of 256^3 particles, K = 64, compensated
// sums: 112.9 -> 104.0 ms at two sinks per lane and two sources a step, 120.1 -> 99.9 at four sinks.
template <int KIND, int MODE, int S, int U, bool KDE, int PAIRS>
__device__ __forceinline__ void accumulate(const float4 (&p)[U], const float (&xi)[S], const float (&yi)[S],
                                           const float (&zi)[S], float c0, float c1, float c2, float e2,
                                           float ib2, float kc, float (&ax)[S], float (&ay)[S], float (&az)[S],
                                           double (&dxs)[S], double (&dys)[S], double (&dzs)[S], float (&rh)[S]) {
    constexpr int G = S * U <= PAIRS ? U : PAIRS / S;   // sources of a group
#pragma unroll
    for (int u0 = 0; u0 < U; u0 += G) {
        float dx[G][S], dy[G][S], dz[G][S], r2[G][S], ri[G][S], gg[G][S];
        unsigned rmin = 0xffffffffu;
#pragma unroll
        for (int u = 0; u < G; u++)
#pragma unroll
            for (int s = 0; s < S; s++) {
                dx[u][s] = p[u0 + u].x - xi[s];
                dy[u][s] = p[u0 + u].y - yi[s];
                dz[u][s] = p[u0 + u].z - zi[s];
                // Plummer: r2 = |d|^2 + eps^2; spline: the guard of coincident pairs
                const float base = KIND == ABACUS_NF_SPLINE ? kTiny : e2;
                r2[u][s] = __builtin_fmaf(dx[u][s], dx[u][s],
                                          __builtin_fmaf(dy[u][s], dy[u][s], __builtin_fmaf(dz[u][s], dz[u][s], base)));
                if constexpr (KIND == ABACUS_NF_SPLINE) rmin = min(rmin, __float_as_uint(r2[u][s]));
            }
        __builtin_amdgcn_s_setprio(3);
#pragma unroll
        for (int u = 0; u < G; u++)
#pragma unroll
            for (int s = 0; s < S; s++) ri[u][s] = __builtin_amdgcn_rsqf(r2[u][s]);
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int u = 0; u < G; u++)
#pragma unroll
            for (int s = 0; s < S; s++) gg[u][s] = (ri[u][s] * ri[u][s]) * ri[u][s];
        if constexpr (KIND == ABACUS_NF_SPLINE) {
            // Spline: g = min(r^-3, c0 + r^2 (c1 r^-1 + c2)).  The cubic force polynomial (divided by r) lies
            // below r^-3 inside eps and above it outside, so the minimum selects the right branch without a
            // compare.  Newtonian regime test for the whole wave: when no lane has a pair closer than eps in
            // this group, g = r^-3 exactly and the polynomial and the minimum are skipped (one wave-uniform
            // branch; close pairs are rare at the softening lengths of the method).  r^2 > 0, so the bit
            // patterns of r^2 order as unsigned integers like the values: half a three-way integer minimum per
            // pair, one compare per group.
            if (__builtin_amdgcn_ballot_w64(rmin < __float_as_uint(e2))) {
                // the constants stay in scalar registers outside this branch (copies hoisted into vector registers
                // cost the main loop spills, whose reloads wait for the chunk being fetched)
                asm volatile("" : "+s"(c0), "+s"(c1), "+s"(c2));
#pragma unroll
                for (int u = 0; u < G; u++)
#pragma unroll
                    for (int s = 0; s < S; s++)
                        gg[u][s] = fminf(gg[u][s], __builtin_fmaf(r2[u][s], __builtin_fmaf(c1, ri[u][s], c2), c0));
            }
        }
#pragma unroll
        for (int u = 0; u < G; u++)
#pragma unroll
            for (int s = 0; s < S; s++) {
                if constexpr (KDE) rh[s] += fmaxf(__builtin_fmaf(-r2[u][s], ib2, kc), 0.f);
                if constexpr (MODE == ABACUS_NF_SUM_FP64) {
                    dxs[s] += (double)(dx[u][s] * gg[u][s]);
                    dys[s] += (double)(dy[u][s] * gg[u][s]);
                    dzs[s] += (double)(dz[u][s] * gg[u][s]);
                } else {
                    ax[s] = __builtin_fmaf(dx[u][s], gg[u][s], ax[s]);
                    ay[s] = __builtin_fmaf(dy[u][s], gg[u][s], ay[s]);
                    az[s] = __builtin_fmaf(dz[u][s], gg[u][s], az[s]);
                }
            }
    }
}

// Twelve floats of a lane to and from LDS (only the lane itself reads them).
template <int S>
__device__ inline void store_low(float4 *p, const float (&x)[S], const float (&y)[S], const float (&z)[S]) {
    if constexpr (S == 4) {
        p[0] = make_float4(x[0], x[1], x[2], x[3]);
        p[1] = make_float4(y[0], y[1], y[2], y[3]);
        p[2] = make_float4(z[0], z[1], z[2], z[3]);
    }
}

template <int S>
__device__ inline void load_low(const float4 *p, float (&x)[S], float (&y)[S], float (&z)[S]) {
    if constexpr (S == 4) {
        const float4 a = p[0], b = p[1], c = p[2];
        x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
        y[0] = b.x; y[1] = b.y; y[2] = b.z; y[3] = b.w;
        z[0] = c.x; z[1] = c.y; z[2] = c.z; z[3] = c.w;
    }
}

// Item of slot j of queue x: the list is dealt to the queues in blocks of kQueueBlock.
__device__ inline int64_t queue_item(int j, int x) {
    return ((int64_t)(j / kQueueBlock) * kQueues + x) * kQueueBlock + j % kQueueBlock;
}

// OCC > 0 asks the compiler for at least OCC waves per SIMD (a register budget of 512/OCC VGPRs), OCC = 0 for four:
// an even number, as the SIMD pairs the plain operations of two waves (at three waves per SIMD one runs unpaired).
template <int KIND, int MODE, int S, int U, int OCC, bool KDE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(OCC > 0 ? OCC : 4, OCC > 0 ? OCC : 8)))
void k_forces(KArgs a) {
    constexpr int NC = KDE ? 4 : 3;  // reduced components per sink: acceleration (+ density)
    // 64 or 80 registers a lane hold neither eight pairs of a group nor, at 64, a chunk under way during the sums
    constexpr int kGroup = OCC > 0 ? kGroupPairs / 2 : kGroupPairs;
    constexpr bool kAhead = OCC < 8;
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = sgpr(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    unsigned char *region = smem + (size_t)wave * a.region;
    float4 *stage = (float4 *)region;
    double *red = (double *)region;
    float *redf = (float *)region;
    ColOff *coff = (ColOff *)(region + (size_t)a.region - kColBytes);
    ColWrap *cwrap = (ColWrap *)(coff + 2 * kMaxCols);
    const int R = a.R;
    const int W = 2 * R + 1;
    const int ncol = W * W;
    const int n_items = a.ws->n_items;
    // Slots of the queue claimed and not yet taken: [jnext, jnext + jleft).  The first slot of every wave is
    // its own number among the waves that start on its queue (the cursors start past those).  Later ones are
    // claimed with one atomic each, or kLightClaim at a time once the queue has reached its light items.  A
    // wave whose queue is drained looks at all cursors with one load before it claims elsewhere: failing
    // claims of every wave on every queue, at 12 ns each on one cache line, were the floor of small calls
    // (32768 particles: 0.48 ms of 0.91).
    int x = blockIdx.x % kQueues;
    int jnext = (int)(blockIdx.x / kQueues) * kWaves + wave, jleft = 1;
    // An item of a whole source list is gone through again for each of its parts.  (A loop over the parts inside saves
    // their set-up but spills twelve registers more of the default kernels, for what it keeps from part to part.)
    int k = n_items, part = 0, parts_left = 0;
    for (;;) {
        if (parts_left == 0) k = n_items;
        while (parts_left == 0) {
            if (jleft == 0) {
                const int want = jnext >= a.ws->light_slot[x] ? kLightClaim : 1;
                int j = 0;
                if (lane == 0) j = atomicAdd(&a.ws->cursor[x][0], want);
                jnext = sgpr(__shfl(j, 0));
                jleft = want;
            }
            const int64_t idx = queue_item(jnext, x);
            jnext++;
            jleft--;
            if (idx < n_items) {
                k = (int)idx;
                break;
            }
            // queue x is drained (its later slots only grow): the next queue with slots left, if any
            jleft = 0;
            int c = INT_MAX;
            if (lane < kQueues) c = __hip_atomic_load(&a.ws->cursor[lane][0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned open = (unsigned)__ballot(lane < kQueues && queue_item(c, lane) < n_items);
            if (!open) break;
            const unsigned turned = (open >> x) | (open << (kQueues - x));   // queue x in bit 0
            x = (x + __builtin_ctz(turned)) % kQueues;
            jnext = __builtin_amdgcn_readlane(c, x);
        }
        if (k >= n_items) break;
        const Item it = a.items[k];
        const int c = sgpr(it.cell);
        const int ib = sgpr(it.box);
        const BoxDev B = a.boxes[ib];
        const ForceBox F = a.fbox[ib];
        const int K = B.K;
        const int lin = c - B.cell_base;
        const int cz = lin % K, cy = (lin / K) % K, cx = lin / (K * K);
        const int cs0 = a.cs[c];
        const int nc = a.cs[c + 1] - cs0;
        const int cell_parts = a.cell_parts[c];   // needed last, fetched with the others
        const TileGeom tg = tile_at(nc, S, a.max_lanes, sgpr(it.tile));
        const int L = tg.L, G = tg.G;
        const int t0 = tg.t0;
        const int nt = tg.nt;
        const int g = lane / L, sub = lane - g * L;

        // sink tile: S sinks per lane, relative to the sink cell centre
        float xi[S], yi[S], zi[S];
#pragma unroll
        for (int s = 0; s < S; s++) {
            const int idx = g * S + s;
            float4 p = make_float4(0.f, 0.f, 0.f, 0.f);
            if (g < G && idx < nt) p = a.spos[cs0 + t0 + idx];
            xi[s] = p.x;
            yi[s] = p.y;
            zi[s] = p.z;
        }

        // the near field, one column per lane, flattened by a prefix sum: source q of column `lane` is slot
        // q + base0, in its second run q + cwrap's base
        ColSeg o;
        o.src0 = o.len0 = o.src1 = o.len1 = 0;
        o.czref0 = o.czref1 = 0.f;
        if (lane < ncol) {
            const int ex = wrap(cx + lane / W - R, K), ey = wrap(cy + lane % W - R, K);
            column_segments(a.cs, B.cell_base + (ex * K + ey) * K, cz, K, R, o);
        }
        int incl = o.len0 + o.len1;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(incl, off);
            if (lane >= off) incl += y;
        }
        const int nsrc = sgpr(__shfl(incl, 63));
        const int cend = incl;                               // end of the column in the flattened list
        const int base0 = o.src0 - (incl - (o.len0 + o.len1));
        const unsigned long long wraps = __ballot(o.len1 > 0);   // columns of two runs
        if (lane < ncol) {
            const float ox = (float)(lane / W - R), oy = (float)(lane % W - R);
            coff[2 * lane] = ColOff{ox, oy, o.czref0};
            coff[2 * lane + 1] = ColOff{ox, oy, o.czref1};
            cwrap[lane] = ColWrap{incl - o.len1, o.src1 - (incl - o.len1)};
        }

        // parts of the source list, nsrc split into P near-equal contiguous ranges (32-bit arithmetic): the item's
        // one, or all of them in turn
        const int split = sgpr(cell_parts);
        const bool whole = split < 0;
        const int P = whole ? -split : split;
        const int pq = nsrc / P, pr = nsrc - pq * P;
        part = whole ? (parts_left > 0 ? part + 1 : 0) : sgpr(it.part);
        parts_left = whole ? P - 1 - part : 0;
        const int j0 = part * pq + min(part, pr);
        const int j1 = j0 + pq + (part < pr ? 1 : 0);

        float ax[S], ay[S], az[S];
        float hx[S], hy[S], hz[S], lx[S], ly[S], lz[S];
        // at four sinks per lane the low words of the compensated sums stay in LDS behind the staged chunk (read
        // and written once per chunk): in registers they would be spilled at four waves per SIMD
        constexpr bool kLowLds = MODE == ABACUS_NF_SUM_COMP32 && S == 4;
        float4 *low = (float4 *)(region + 64 * kRounds * sizeof(float4)) + 3 * lane;
        double dxs[S], dys[S], dzs[S];
        float rh[S];
        double rhd[S];
#pragma unroll
        for (int s = 0; s < S; s++) {
            ax[s] = ay[s] = az[s] = 0.f;
            hx[s] = hy[s] = hz[s] = lx[s] = ly[s] = lz[s] = 0.f;
            dxs[s] = dys[s] = dzs[s] = 0.0;
            rh[s] = 0.f;
            rhd[s] = 0.0;
        }
        const float c0 = uniform(F.c0), c1 = uniform(F.c1), c2 = uniform(F.c2), e2 = uniform(F.eps2);
        const float ib2 = uniform(F.kde_ib2), kc = uniform(F.kde_c);
        const int step = L * U;
        const int nmax = (a.chunk / step) * step;

        // A chunk [f, f + n) of the flattened source list is fetched into registers with all of its loads in
        // flight at once: slot 64 r + lane in v[r], its run of a column in byte r of runs (255: none).  The chunk
        // after the one being summed is under way during the sums.
        float4 v[kRounds];
        static_assert(kRounds == 4 && 2 * kMaxCols < 255, "a byte per round");
        unsigned runs = 0xffffffffu;
        int ci = 0;   // first column that reaches past the chunk fetched last
        auto fetch = [&](int f, int n) {
            int src[kRounds], w[kRounds];
#pragma unroll
            for (int r = 0; r < kRounds; r++) {
                src[r] = 0;
                w[r] = 255;
            }
            const int stop = f + n;
            for (;; ci++) {
                const int e = __builtin_amdgcn_readlane(cend, ci);
                if (e > f) {
                    const int b0 = __builtin_amdgcn_readlane(base0, ci);
                    const int b = e > stop ? stop : e;
                    if (!((wraps >> ci) & 1)) {   // one run
#pragma unroll
                        for (int r = 0; r < kRounds; r++) {
                            const int q = f + 64 * r + lane;
                            if (w[r] == 255 && q < b) {
                                src[r] = q + b0;
                                w[r] = 2 * ci;
                            }
                        }
                    } else {        // the column wraps through the box boundary
                        const ColWrap cw = cwrap[ci];
                        const int m = cw.split, b1 = cw.base;
#pragma unroll
                        for (int r = 0; r < kRounds; r++) {
                            const int q = f + 64 * r + lane;
                            if (w[r] == 255 && q < b) {
                                src[r] = q + (q < m ? b0 : b1);
                                w[r] = 2 * ci + (q < m ? 0 : 1);
                            }
                        }
                    }
                }
                if (e >= stop || ci + 1 >= ncol) break;
            }
#pragma unroll
            for (int r = 0; r < kRounds; r++)
                if (w[r] != 255) v[r] = a.spos[src[r]];
            runs = (unsigned)w[0] | (unsigned)w[1] << 8 | (unsigned)w[2] << 16 | (unsigned)w[3] << 24;
        };
        if constexpr (kLowLds) store_low(low, lx, ly, lz);
        wave_lds_sync();   // the column tables
        if (j0 < j1) fetch(j0, min(nmax, j1 - j0));

        for (int f = j0; f < j1;) {
            const int n = min(nmax, j1 - f);
            const int npad = ((n + step - 1) / step) * step;
            // stage the chunk with the cell offsets applied; the last step is filled up with far sources
#pragma unroll
            for (int r = 0; r < kRounds; r++) {
                const int q = 64 * r + lane;
                const int run = (runs >> (8 * r)) & 255;
                if (run != 255) {
                    const ColOff co = coff[run];
                    stage[q] = make_float4(v[r].x + co.x, v[r].y + co.y, v[r].z + (v[r].w - co.czref), 0.f);
                } else if (q < npad) {
                    stage[q] = make_float4(kFar, kFar, kFar, 0.f);
                }
            }
            if (kAhead && f + n < j1) fetch(f + n, min(nmax, j1 - f - n));
            wave_lds_sync();

            if constexpr (MODE == ABACUS_NF_SUM_COMP32) {
#pragma unroll
                for (int s = 0; s < S; s++) ax[s] = ay[s] = az[s] = 0.f;
            }
            // uniform trip count; one sink group per lane (L == 1) reads with immediate LDS offsets
            const int iters = npad / step;
            if (L == 1) {
                const float4 *sp = stage;
                for (int it = 0; it < iters; ++it) {
                    float4 p[U];
#pragma unroll
                    for (int u = 0; u < U; u++) p[u] = sp[u];
                    sp += U;
                    accumulate<KIND, MODE, S, U, KDE, kGroup>(p, xi, yi, zi, c0, c1, c2, e2, ib2, kc, ax, ay, az, dxs, dys,
                                                      dzs, rh);
                }
            } else {
                const float4 *sp = stage + sub;
                for (int it = 0; it < iters; ++it) {
                    float4 p[U];
#pragma unroll
                    for (int u = 0; u < U; u++) p[u] = sp[u * L];
                    sp += step;
                    accumulate<KIND, MODE, S, U, KDE, kGroup>(p, xi, yi, zi, c0, c1, c2, e2, ib2, kc, ax, ay, az, dxs, dys,
                                                      dzs, rh);
                }
            }
            if constexpr (KDE && MODE != ABACUS_NF_SUM_FP32) {
#pragma unroll
                for (int s = 0; s < S; s++) {
                    rhd[s] += (double)rh[s];
                    rh[s] = 0.f;
                }
            }
            if constexpr (MODE == ABACUS_NF_SUM_COMP32) {
                if constexpr (kLowLds) load_low(low, lx, ly, lz);
#pragma unroll
                for (int s = 0; s < S; s++) {
                    float e;
                    two_sum(hx[s], ax[s], hx[s], e);
                    lx[s] += e;
                    two_sum(hy[s], ay[s], hy[s], e);
                    ly[s] += e;
                    two_sum(hz[s], az[s], hz[s], e);
                    lz[s] += e;
                }
                if constexpr (kLowLds) store_low(low, lx, ly, lz);
            }
            if (!kAhead && f + n < j1) fetch(f + n, min(nmax, j1 - f - n));
            wave_lds_sync();
            f += n;
        }

        if constexpr (kLowLds) {
            load_low(low, lx, ly, lz);
            wave_lds_sync();
        }
        // Ordered reduction over the L lanes that share each sink: every lane leaves its sums in LDS, lane o of
        // the G S NC totals adds the L parts of total o in lane order, in place of the first of them.
#pragma unroll
        for (int s = 0; s < S; s++) {
            const int o = (lane * S + s) * NC;
            if constexpr (MODE == ABACUS_NF_SUM_FP32) {
                redf[o + 0] = ax[s];
                redf[o + 1] = ay[s];
                redf[o + 2] = az[s];
                if constexpr (KDE) redf[o + 3] = rh[s];
            } else if constexpr (MODE == ABACUS_NF_SUM_COMP32) {
                red[o + 0] = (double)hx[s] + (double)lx[s];
                red[o + 1] = (double)hy[s] + (double)ly[s];
                red[o + 2] = (double)hz[s] + (double)lz[s];
                if constexpr (KDE) red[o + 3] = rhd[s];
            } else {
                red[o + 0] = dxs[s];
                red[o + 1] = dys[s];
                red[o + 2] = dzs[s];
                if constexpr (KDE) red[o + 3] = rhd[s];
            }
        }
        wave_lds_sync();
        if (L > 1) {
            for (int o = lane; o < G * S * NC; o += 64) {
                const int first = (o / (S * NC)) * (L - 1) * S * NC + o;
                if constexpr (MODE == ABACUS_NF_SUM_FP32) {
                    float t = 0.f;
                    for (int q = 0; q < L; q++) t += redf[first + q * S * NC];
                    redf[first] = t;
                } else {
                    double t = 0.0;
                    for (int q = 0; q < L; q++) t += red[first + q * S * NC];
                    red[first] = t;
                }
            }
            wave_lds_sync();
        }
        // A whole list's parts are added up in order in the sink's slot, as k_finalize adds those of a split one.
        const bool done = P <= 1 || (whole && part + 1 == P);
        double amax2 = 0.0;   // largest |a|^2 this lane writes (cells written here, not split ones)
        for (int idx = lane; idx < nt; idx += 64) {
            const int base = ((idx / S) * L * S + idx % S) * NC;
            double *slot = nullptr;
            if (P > 1) slot = a.partials + (int64_t)NC * (a.cell_pbase[c] + (int64_t)(whole ? 0 : part) * nc + t0 + idx);
            if (whole) {
#pragma unroll
                for (int d = 0; d < NC; d++) {
                    if constexpr (MODE == ABACUS_NF_SUM_FP32)
                        redf[base + d] = (part > 0 ? (float)slot[d] : 0.f) + redf[base + d];
                    else
                        red[base + d] = (part > 0 ? slot[d] : 0.0) + red[base + d];
                }
            }
            if (done) {
                const int64_t i = a.perm[cs0 + t0 + idx];
                double wr[3];   // the values written
#pragma unroll
                for (int d = 0; d < NC; d++) {
                    double val;   // the value before its (optional) rounding to FP32
                    if constexpr (MODE == ABACUS_NF_SUM_FP32) {
                        const float t = redf[base + d];
                        val = d < 3 ? t * F.scalef : t;
                    } else {
                        const double t = red[base + d];
                        val = d < 3 ? t * F.scale : t;
                    }
                    if (d == 3) {
                        a.rho[i] = (float)val;
                    } else if (a.acc64) {
                        a.acc64[3 * i + d] = val;
                        wr[d] = val;
                    } else {
                        a.acc[3 * i + d] = (float)val;
                        wr[d] = (double)(float)val;
                    }
                }
                const double m = norm2_written(wr[0], wr[1], wr[2]);
                amax2 = m > amax2 ? m : amax2;
            } else {
#pragma unroll
                for (int d = 0; d < NC; d++) {
                    if constexpr (MODE == ABACUS_NF_SUM_FP32)
                        slot[d] = redf[base + d];
                    else
                        slot[d] = red[base + d];
                }
            }
        }
        if (done) {   // per-cell maximum of |a|^2 (the input of the step-size criterion)
            amax2 = wave_max_f64(amax2);
            if (lane == 0 && amax2 > 0.0) cell_max(a.amax, c, amax2);
        }
        wave_lds_sync();
    }
}

// Sinks whose source list was split over items: add the parts in order and write the result.
template <int MODE, int NC>
__global__ __launch_bounds__(256) void k_finalize(const WorkState *__restrict__ ws, int64_t partial_capacity,
                                                  const int32_t *__restrict__ keys, const int32_t *__restrict__ cs,
                                                  const int32_t *__restrict__ perm,
                                                  const int32_t *__restrict__ cell_parts,
                                                  const int64_t *__restrict__ cell_pbase,
                                                  const double *__restrict__ partials,
                                                  const BoxDev *__restrict__ boxes, int n_boxes,
                                                  const ForceBox *__restrict__ fbox, float *__restrict__ acc,
                                                  double *__restrict__ acc64, float *__restrict__ rho,
                                                  unsigned long long *__restrict__ amax, int64_t n) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (ws->overflow) return;
    const int lane = threadIdx.x & 63;
    int32_t c = -1;
    int P = 0;
    double m = 0.0;   // |a|^2 written for this slot
    if (s < n) {
        c = keys[s];
        P = cell_parts[c];
    }
    if (!__ballot(P > 1)) return;   // most waves of a large box: no split cell
    if (s < n) {
        const int cs0 = cs[c], nc = cs[c + 1] - cs0;
        const int64_t base = P > 1 ? cell_pbase[c] + (s - cs0) : 0;
        if (P > 1 && base + (int64_t)(P - 1) * nc < partial_capacity) {
            const int b = n_boxes > 1 ? box_of_cell(boxes, n_boxes, c) : 0;
            const ForceBox F = fbox[b];
            const int64_t i = perm[s];
            double w[3];
            for (int d = 0; d < NC; d++) {
                double v;   // the value before its (optional) rounding to FP32
                if constexpr (MODE == ABACUS_NF_SUM_FP32) {
                    float t = 0.f;
#pragma unroll 8
                    for (int p = 0; p < P; p++) t += (float)partials[NC * (base + (int64_t)p * nc) + d];
                    v = d < 3 ? t * F.scalef : t;
                } else {
                    double t = 0.0;
#pragma unroll 8
                    for (int p = 0; p < P; p++) t += partials[NC * (base + (int64_t)p * nc) + d];
                    v = d < 3 ? t * F.scale : t;
                }
                if (d == 3) {
                    rho[i] = (float)v;
                } else if (acc64) {
                    acc64[3 * i + d] = v;
                    w[d] = v;
                } else {
                    acc[3 * i + d] = (float)v;
                    w[d] = (double)(float)v;
                }
            }
            m = norm2_written(w[0], w[1], w[2]);
        }
    }
    // per-cell maximum over the wave's slots: a segmented max-scan (slots are sorted by cell, so equal
    // keys are adjacent) and one update by the last lane of each run
    for (int off = 1; off < 64; off <<= 1) {
        const double y = __shfl_up(m, off);
        const int cy = __shfl_up(c, off);
        if (lane >= off && cy == c) m = m > y ? m : y;
    }
    const int cn = __shfl_down(c, 1);
    if (c >= 0 && m > 0.0 && (lane == 63 || cn != c)) cell_max(amax, c, m);
}

// ---------------------------------------------------------------- variant dispatch

typedef void (*ForcesKernel)(KArgs);

template <int KIND, int MODE, int S, int U, bool KDE>
ForcesKernel pick_occ(int occ) {
    if constexpr (KDE) {  // density variants: compiler's register budget, 6 or 8 waves per SIMD
        switch (occ) {
            case 6: return k_forces<KIND, MODE, S, U, 6, true>;
            case 8: return k_forces<KIND, MODE, S, U, 8, true>;
            default: return k_forces<KIND, MODE, S, U, 0, true>;
        }
    } else {
        switch (occ) {
            case 6: return k_forces<KIND, MODE, S, U, 6, false>;
            case 8: return k_forces<KIND, MODE, S, U, 8, false>;
            default: return k_forces<KIND, MODE, S, U, 0, false>;
        }
    }
}

template <int KIND, int MODE, int S, bool KDE>
ForcesKernel pick_u(int U, int occ) {
    switch (U) {
        case 1: return pick_occ<KIND, MODE, S, 1, KDE>(occ);
        case 4:
            if constexpr (!KDE) return pick_occ<KIND, MODE, S, 4, KDE>(occ);
            else return pick_occ<KIND, MODE, S, 2, KDE>(occ);
        default: return pick_occ<KIND, MODE, S, 2, KDE>(occ);
    }
}

template <int KIND, int MODE, bool KDE>
ForcesKernel pick_s(int S, int U, int occ) {
    switch (S) {
        case 1: return pick_u<KIND, MODE, 1, KDE>(U, occ);
        case 4: return pick_u<KIND, MODE, 4, KDE>(U, occ);
        default: return pick_u<KIND, MODE, 2, KDE>(U, occ);
    }
}

template <int KIND, bool KDE>
ForcesKernel pick_mode(int mode, int S, int U, int occ) {
    switch (mode) {
        case ABACUS_NF_SUM_COMP32: return pick_s<KIND, ABACUS_NF_SUM_COMP32, KDE>(S, U, occ);
        case ABACUS_NF_SUM_FP64: return pick_s<KIND, ABACUS_NF_SUM_FP64, KDE>(S, U, occ);
        default: return pick_s<KIND, ABACUS_NF_SUM_FP32, KDE>(S, U, occ);
    }
}

ForcesKernel pick_kernel(abacus_nf_kind kind, abacus_nf_sum mode, int S, int U, int occ, bool kde) {
    if (kde)
        return kind == ABACUS_NF_PLUMMER ? pick_mode<ABACUS_NF_PLUMMER, true>(mode, S, U, occ)
                                         : pick_mode<ABACUS_NF_SPLINE, true>(mode, S, U, occ);
    return kind == ABACUS_NF_PLUMMER ? pick_mode<ABACUS_NF_PLUMMER, false>(mode, S, U, occ)
                                     : pick_mode<ABACUS_NF_SPLINE, false>(mode, S, U, occ);
}

// Sources staged at a time: the tuning's chunk, as far as the registers of a fetch hold it.
int staged_chunk(const abacus_nf_tuning &t) { return t.chunk < 64 * kRounds ? t.chunk : 64 * kRounds; }

size_t region_bytes(const abacus_nf_tuning &t) {
    size_t stage = (size_t)staged_chunk(t) * sizeof(float4);
    size_t red = (size_t)64 * t.sinks_per_lane * 4 * sizeof(double);
    // the low words of the compensated sums at four sinks per lane lie behind a full chunk
    const size_t low = t.sinks_per_lane == 4 ? 64 * (kRounds * sizeof(float4) + 3 * sizeof(float4)) : 0;
    size_t main = std::max(std::max(stage, red), low);
    return (main + kColBytes + 15) & ~(size_t)15;
}

}  // namespace

// ---------------------------------------------------------------- host side

hipError_t launch_set_force_boxes(const double *eps, const double *gm, const double *kde_b, abacus_nf_kind kind,
                                  const abacus_nf_box *boxes, int n_boxes, ForceBox *dst, const ForcesArgs &a,
                                  hipStream_t st) {
    for (int first = 0; first < n_boxes; first += kFBoxChunk) {
        FBoxChunk ch;
        memset(&ch, 0, sizeof(ch));
        ch.first = first;
        ch.count = n_boxes - first < kFBoxChunk ? n_boxes - first : kFBoxChunk;
        for (int k = 0; k < ch.count; k++) {
            const int b = first + k;
            const double w = boxes[b].box / boxes[b].K;
            const double e = eps[b] / w;
            ForceBox &f = ch.f[k];
            f.c0 = (float)(10.0 / (e * e * e));
            f.c1 = (float)(-15.0 / (e * e * e * e));
            f.c2 = (float)(6.0 / (e * e * e * e * e));
            f.eps2 = (float)(e * e);
            f.scale = gm[b] / (w * w);
            f.scalef = (float)f.scale;
            if (kde_b) {
                const double bc = kde_b[b] / w;
                const double ib2 = 1.0 / (bc * bc);
                const double offset = kind == ABACUS_NF_PLUMMER ? (double)f.eps2 : (double)kTiny;
                f.kde_ib2 = (float)ib2;
                f.kde_c = (float)(1.0 + offset * ib2);
            } else {
                f.kde_ib2 = 0.f;
                f.kde_c = 0.f;
            }
            f.pad = 0;
        }
        hipLaunchKernelGGL(k_set_fbox, dim3(1), dim3(64), 0, st, ch, dst, a.ws, a.wb, a.grid);
        hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

namespace {

hipError_t launch_cells(const ForcesArgs &a, bool clear_amax, hipStream_t st) {
    if (a.n_cells <= 0) return hipSuccess;
    // at most 2048 workgroups (eight per CU), so that their additions to a box's totals stay few
    const unsigned g = grid_for(a.n_cells, 256);
    auto k = a.R == 1 ? k_wl_cells<1> : (a.R == 2 ? k_wl_cells<2> : k_wl_cells<3>);
    hipLaunchKernelGGL(k, dim3(g < 2048 ? g : 2048), dim3(256), 0, st, a.cell_start, a.boxes, a.n_boxes, a.n_cells,
                       a.tune.sinks_per_lane, a.tune.max_lanes, a.cell_nsrc, clear_amax ? a.amax : nullptr, a.wb);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_count_interactions(const ForcesArgs &a, hipStream_t st) {
    hipLaunchKernelGGL(k_wl_clear, dim3(1), dim3(64), 0, st, a.ws, a.wb, a.n_boxes);
    const hipError_t e = hipGetLastError();
    return e != hipSuccess ? e : launch_cells(a, false, st);
}

hipError_t build_work_list(const ForcesArgs &a, hipStream_t st) {
    hipError_t e = launch_cells(a, true, st);
    if (e != hipSuccess || a.n_cells <= 0) return e;
    const int S = a.tune.sinks_per_lane, ML = a.tune.max_lanes;
    const unsigned gc = grid_for(a.n_cells, 256);
    hipLaunchKernelGGL(k_wl_plan, dim3(grid_for(a.n_boxes, 256)), dim3(256), 0, st, a.ws, a.wb, a.boxes, a.n_boxes, S,
                       a.tune.part_sources);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (a.short_room) {
        hipLaunchKernelGGL(k_wl_bins, dim3(gc), dim3(256), 0, st, a.cell_start, a.cell_nsrc, a.boxes, a.n_boxes,
                           a.n_cells, S, ML, a.tune.part_sources, a.wb, a.ws);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(k_wl_fit, dim3(1), dim3(64), 0, st, a.ws, a.partial_capacity, a.item_capacity);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_wl_count, dim3(gc), dim3(256), 0, st, a.cell_start, a.cell_nsrc, a.boxes, a.n_boxes,
                       a.n_cells, S, ML, a.tune.part_sources, a.wb, a.ws, a.cell_parts, a.cell_pbase);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    // few cells have many items each: fewer cells to a workgroup then
    const int per_block = a.n_cells >= 16384 ? 256 : 16;
    hipLaunchKernelGGL(k_wl_emit, dim3(grid_for(a.n_cells, per_block)), dim3(256), 0, st, a.cell_start, a.cell_nsrc,
                       a.cell_parts, a.boxes, a.n_boxes, a.n_cells, S, ML, a.ws, a.items, a.item_capacity,
                       a.partial_capacity, per_block, a.err);
    return hipGetLastError();
}

int forces_grid(const abacus_nf_tuning &t, abacus_nf_kind kind, abacus_nf_sum mode, bool kde, int device) {
    ForcesKernel kfn = pick_kernel(kind, mode, t.sinks_per_lane, t.unroll, t.occupancy, kde);
    const size_t lds = region_bytes(t) * kWaves;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kfn, kThreads, lds) != hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    if (t.waves_per_cu > 0) {
        int want = (t.waves_per_cu + kWaves - 1) / kWaves;
        if (want < per_cu) per_cu = want;
    }
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) cus = 1;
    return per_cu * cus;
}

hipError_t launch_forces(const ForcesArgs &a, hipStream_t st) {
    if (a.n_total <= 0) return hipSuccess;
    KArgs k;
    k.spos = a.spos;
    k.cs = a.cell_start;
    k.perm = a.perm;
    k.items = a.items;
    k.ws = a.ws;
    k.boxes = a.boxes;
    k.fbox = a.fbox;
    k.cell_parts = a.cell_parts;
    k.cell_pbase = a.cell_pbase;
    k.partials = a.partials;
    k.acc = a.acc;
    k.acc64 = a.acc64;
    k.rho = a.rho;
    k.amax = a.amax;
    k.R = a.R;
    k.chunk = staged_chunk(a.tune);
    k.max_lanes = a.tune.max_lanes;
    k.region = (int)region_bytes(a.tune);
    ForcesKernel kfn = pick_kernel(a.kind, a.mode, a.tune.sinks_per_lane, a.tune.unroll, a.tune.occupancy,
                                   a.rho != nullptr);
    hipLaunchKernelGGL(kfn, dim3(a.grid), dim3(kThreads), (size_t)k.region * kWaves, st, k);
    return hipGetLastError();
}

hipError_t launch_finalize(const ForcesArgs &a, hipStream_t st) {
    if (a.n_total <= 0) return hipSuccess;
    const unsigned gn = grid_for(a.n_total, 256);
    const bool f32 = a.mode == ABACUS_NF_SUM_FP32, kde = a.rho != nullptr;
    auto kfn = f32 ? (kde ? k_finalize<ABACUS_NF_SUM_FP32, 4> : k_finalize<ABACUS_NF_SUM_FP32, 3>)
                   : (kde ? k_finalize<ABACUS_NF_SUM_FP64, 4> : k_finalize<ABACUS_NF_SUM_FP64, 3>);
    hipLaunchKernelGGL(kfn, dim3(gn), dim3(256), 0, st, a.ws, a.partial_capacity, a.keys, a.cell_start, a.perm,
                       a.cell_parts, a.cell_pbase, a.partials, a.boxes, a.n_boxes, a.fbox, a.acc, a.acc64, a.rho,
                       a.amax, a.n_total);
    return hipGetLastError();
}

}  // namespace anf
