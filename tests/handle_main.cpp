// The library's host side (csrc/api.hip, host code alone) against a stand-in for the HIP runtime and the launchers, for
// the host-side test of handles when device memory runs out.  Device allocations are numbers; a launcher that is
// handed a null pointer it would read or write says so.
#include <cstdio>
#include <cstring>
#include <map>
#include <vector>

#include "../paper_2110_11398_amd/csrc/nf_internal.h"

static size_t budget = 0, used = 0;
static std::map<char *, size_t> live;
static char *next_address = (char *)0x100000;
static bool null_pointer = false;
static int allocations = 0;
static anf::ForcesArgs last_forces;

extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) {
    if (used + bytes > budget) return hipErrorOutOfMemory;
    used += bytes;
    allocations++;
    live[next_address] = bytes;
    *p = next_address;
    next_address += (bytes + 4095) / 4096 * 4096;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    auto it = live.find((char *)p);
    if (it == live.end()) return hipErrorInvalidValue;
    used -= it->second;
    live.erase(it);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemcpy(void *dst, const void *, size_t n, hipMemcpyKind) {
    memset(dst, 0, n);   // the device error word
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t) {
    if (!src || !dst) null_pointer = true;
    if (kind == hipMemcpyDeviceToHost) memset(dst, 0, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
}

namespace anf {
static hipError_t need(std::initializer_list<const void *> ps) {
    for (const void *p : ps)
        if (!p) null_pointer = true;
    return hipSuccess;
}
int forces_grid(const abacus_nf_tuning &, abacus_nf_kind, abacus_nf_sum, bool, int) { return 1024; }
hipError_t launch_kick(float *, const float *, int64_t, const BoxDev *b, int, const double *d, int, hipStream_t) { return need({b, d}); }
hipError_t launch_drift(float *, const float *, int64_t, const BoxDev *b, int, const double *d, int, hipStream_t) { return need({b, d}); }
hipError_t sort_by_cell(const SortArgs &a, int, int32_t **keys, bool *starts, hipStream_t) {
    *keys = a.keys_a;
    *starts = true;
    return need({a.boxes, a.keys_a, a.keys_b, a.perm, a.pay, a.spos, a.cell_start, a.temp, a.err});
}
hipError_t plan(const ForcesArgs &a) {
    last_forces = a;
    return need({a.spos, a.cell_start, a.perm, a.keys, a.boxes, a.fbox, a.items, a.ws, a.wb, a.cell_nsrc, a.cell_parts,
                 a.cell_pbase, a.partials, a.amax});
}
hipError_t launch_forces(const ForcesArgs &a, hipStream_t) { return plan(a); }
hipError_t build_work_list(const ForcesArgs &a, hipStream_t) { return plan(a); }
hipError_t launch_finalize(const ForcesArgs &a, hipStream_t) { return plan(a); }
hipError_t launch_count_interactions(const ForcesArgs &a, hipStream_t) { return plan(a); }
hipError_t launch_taylor(const float4 *s, const int32_t *k, const int32_t *p, const BoxDev *b, int, int64_t, int64_t, int,
                         const double *, float *, int, hipStream_t) { return need({s, k, p, b}); }
hipError_t launch_reorder(float *const *, int, int64_t *, int32_t *p, int64_t, void *t, int, hipStream_t) { return need({p, t}); }
hipError_t launch_fill_u64(unsigned long long *p, int64_t, unsigned long long, hipStream_t) { return need({p}); }
hipError_t launch_timestep(const float *, const float *, const unsigned long long *, const int32_t *k, const int32_t *p,
                           const int32_t *c, const BoxDev *b, int, int64_t, double *w, unsigned long long *m,
                           hipStream_t) { return need({k, p, c, b, w, m}); }
size_t scan_temp_bytes(int64_t n) { return n; }
hipError_t launch_set_boxes(const abacus_nf_box *, int, const int32_t *, BoxDev *d, hipStream_t) { return need({d}); }
int taylor_max_order() { return 10; }
int multipole_max_order() { return 10; }
hipError_t launch_cell_start(const int32_t *k, int64_t, int64_t, int32_t *e, int32_t *c, void *, hipStream_t) { return need({k, e, c}); }
hipError_t launch_multipoles(const float4 *s, const int32_t *k, const int32_t *c, const BoxDev *b, int, int64_t, int64_t,
                             int, const double *, double *m, double *p, double *, int, hipStream_t) { return need({s, k, c, b, m, p}); }
size_t timestep_min_words(int n) { return 64 * (size_t)n; }
size_t timestep_min_offset(int) { return 0; }
size_t timestep_partial_doubles(int64_t n) { return n; }
size_t multipole_partial_doubles(int64_t n, int) { return n; }
hipError_t upload_box_doubles(const double *, int, double *d, hipStream_t) { return need({d}); }
hipError_t launch_set_force_boxes(const double *, const double *, const double *, abacus_nf_kind, const abacus_nf_box *, int,
                                  ForceBox *d, const ForcesArgs &a, hipStream_t) { return need({d, a.ws, a.wb}); }
}  // namespace anf

static float fake[4];
static const double one[1] = {0.01};
static float *const arrays[1] = {fake};

static int build(abacus_nf_cells *h, int64_t n, int K) {
    abacus_nf_box b{};
    b.n = n;
    b.box = 1.0;
    b.K = K;
    return abacus_nf_build_cells(fake, n, &b, 1, 2, nullptr, h);
}

static int forces(abacus_nf_cells h) { return abacus_nf_forces(h, one, ABACUS_NF_SPLINE, one, ABACUS_NF_SUM_FP32, fake, nullptr); }

// every call that reads a built handle
static void use(const char *what, abacus_nf_cells h) {
    null_pointer = false;
    double dt[1];
    int64_t a = 0, b = 0;
    const int rc[] = {forces(h),
                      abacus_nf_forces_f64(h, one, ABACUS_NF_SPLINE, one, ABACUS_NF_SUM_FP32, dt, nullptr),
                      abacus_nf_forces_density(h, one, ABACUS_NF_SPLINE, one, ABACUS_NF_SUM_FP32, one, fake, fake, nullptr),
                      abacus_nf_multipoles(h, 2, one, dt, nullptr),
                      abacus_nf_taylor_forces(h, 2, dt, fake, nullptr),
                      abacus_nf_timestep(h, fake, fake, 0.25, dt, nullptr),
                      abacus_nf_timestep(h, fake, nullptr, 0.25, dt, nullptr),
                      abacus_nf_reorder(h, arrays, 1, nullptr, nullptr),
                      abacus_nf_interactions(h, nullptr, &a),
                      abacus_nf_cells_size(h, &a, &b),
                      abacus_nf_kick(h, one, fake, fake, nullptr),
                      abacus_nf_kdk_step(h, one, one, ABACUS_NF_SPLINE, one, ABACUS_NF_SUM_FP32, fake, fake, fake, nullptr),
                      abacus_nf_drift(h, one, fake, fake, nullptr)};
    printf("%s", what);
    for (int r : rc) printf(" %d", r);
    printf(" null=%d\n", (int)null_pointer);
}

int main() {
    abacus_nf_cells h = nullptr;
    budget = (size_t)1 << 40;
    printf("build %d\n", build(&h, 1000, 5));
    use("built", h);
    printf("build %d\n", build(&h, 1000, 5));
    budget = used + (1 << 20);
    printf("grow %d\n", build(&h, 1000000, 50));
    use("failed", h);
    budget = (size_t)1 << 40;
    printf("build %d\n", build(&h, 1000000, 50));
    // lists: as wanted, the least ones, none
    const anf::ListRoom want = anf::list_room(1000000, 125000, 1), least = anf::least_room(1000000, 125000);
    const size_t cells = 125000 * (size_t)24 + (1 << 20), before = used;
    for (size_t slots : {want.slots, least.slots, least.slots / 2}) {
        // a fresh handle's lists each time
        printf("build %d", build(&h, 1000000, 50));
        abacus_nf_tuning t;
        abacus_nf_get_tuning(h, &t);
        t.item_capacity = 1000 + (int64_t)slots % 7;
        abacus_nf_set_tuning(h, &t);
        budget = before + cells + 32 * slots;
        null_pointer = false;
        const int rc = forces(h);
        printf(" forces %d", rc);
        if (rc == ABACUS_NF_OK)
            printf(" slots %lld short %d", (long long)last_forces.partial_capacity, (int)last_forces.short_room);
        budget = (size_t)1 << 40;
        printf(" again %d null=%d\n", forces(h), (int)null_pointer);
    }
    printf("want %lld least %lld\n", (long long)want.slots, (long long)least.slots);
    // sinks per lane of the summation modes: by default, set, by default again, and with few lanes
    for (int set : {0, 4, 1, -1, -8}) {
        abacus_nf_tuning t;
        abacus_nf_get_tuning(h, &t);
        t.item_capacity = 0;
        t.sinks_per_lane = set > 0 ? set : 0;
        if (set == -8) t.max_lanes = 8;
        abacus_nf_set_tuning(h, set == -1 ? nullptr : &t);
        printf("sinks");
        for (abacus_nf_sum mode : {ABACUS_NF_SUM_FP32, ABACUS_NF_SUM_COMP32, ABACUS_NF_SUM_FP64}) {
            abacus_nf_forces(h, one, ABACUS_NF_SPLINE, one, mode, fake, nullptr);
            printf(" %d", last_forces.tune.sinks_per_lane);
        }
        abacus_nf_get_tuning(h, &t);
        printf(" get %d\n", t.sinks_per_lane);
    }
    // smaller calls on the handle of a batch: fewer boxes of the same totals, fewer particles and cells
    abacus_nf_set_tuning(h, nullptr);
    for (int pass = 0; pass < 2; pass++)
        for (int n_boxes : {8, 4, 2, 1, 3}) {
            std::vector<abacus_nf_box> b(n_boxes);
            std::vector<double> v(n_boxes, 0.01);
            const int64_t n = 840000 / n_boxes, odd = pass ? 17 : 0;
            const int K = n_boxes == 8 ? 40 : n_boxes == 3 ? 20 : 50;
            for (int i = 0; i < n_boxes; i++) {
                b[i] = abacus_nf_box{};
                b[i].offset = i * (n - odd);
                b[i].n = n - odd;
                b[i].box = 1.0;
                b[i].K = K;
            }
            allocations = 0;
            int rc = abacus_nf_build_cells(fake, n_boxes * (n - odd), b.data(), n_boxes, 2, nullptr, &h);
            if (rc == 0) rc = abacus_nf_forces(h, v.data(), ABACUS_NF_SPLINE, v.data(), ABACUS_NF_SUM_FP32, fake, nullptr);
            printf("boxes %d rc %d allocations %d\n", n_boxes, rc, allocations);
        }
    abacus_nf_free_cells(h);
    return 0;
}
