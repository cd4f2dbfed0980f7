/* The library's host code on a HIP runtime made of host memory, with every
 * allocation of a call failing in turn; who writes a read-out's arrays; and the
 * order of a step's tiles.
 *
 * The HIP calls that lbm_runtime.cpp and lbm_pool.cpp make are defined here:
 * device and pinned memory come from malloc and are kept in a table, copies
 * check that their device side lies in it, work happens at once.  The kernel
 * launches check their pointers against the table and write what the host
 * reads back.  One chosen allocation (hipMalloc or hipHostMalloc) fails with
 * hipErrorOutOfMemory; as on a GPU that error stays the thread's last error
 * until hipGetLastError takes it, which every launch here ends with.
 *
 * Test infrastructure: tests/test_pool_allocation.py compiles this with both
 * sources and the sanitizers and runs it on the CPU. */
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "lbm.h"
#include "lbm_host.h"
#include "lbm_internal.h"

static int failures = 0;
static std::string where;
#define EXPECT(cond)                                                                         \
    do {                                                                                     \
        if (!(cond)) {                                                                       \
            fprintf(stderr, "%d [%s]: expectation failed: %s (%s)\n", __LINE__, where.c_str(), #cond, \
                    lbm_last_error());                                                       \
            ++failures;                                                                      \
        }                                                                                    \
    } while (0)

/* ---- the runtime ------------------------------------------------------------ */
struct Block {
    size_t bytes;
    bool host;
};
static std::map<char*, Block> blocks;
static long allocs = 0, fail_at = -1, frees = 0;
static hipError_t last = hipSuccess;
static bool busy = false;             // the work enqueued last has not ended
static lbmk::Moments told;            // where the last read-out's kernel wrote
static int copies = 0;                // device to host

static const std::pair<char* const, Block>* find(const void* p) {
    auto it = blocks.upper_bound((char*)p);
    if (it == blocks.begin()) return nullptr;
    --it;
    return (char*)p < it->first + it->second.bytes ? &*it : nullptr;
}
static bool holds(const void* p, size_t bytes) {
    const auto* b = find(p);
    return b && (size_t)((char*)p - b->first) + bytes <= b->second.bytes;
}
static hipError_t result(hipError_t e) {
    if (e != hipSuccess) last = e;
    return e;
}
static hipError_t take(void** out, size_t bytes, bool host) {
    if (allocs++ == fail_at) return result(hipErrorOutOfMemory);
    char* p = (char*)malloc(bytes);
    blocks[p] = {bytes, host};
    *out = p;
    return hipSuccess;
}
static hipError_t give(void* p, bool host) {
    if (!p) return hipSuccess;
    auto it = blocks.find((char*)p);
    EXPECT(it != blocks.end() && it->second.host == host);
    if (it == blocks.end()) return result(hipErrorInvalidValue);
    free(it->first);
    blocks.erase(it);
    ++frees;
    return hipSuccess;
}

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return take(p, n, false); }
hipError_t hipFree(void* p) { return give(p, false); }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return take(p, n, true); }
hipError_t hipHostFree(void* p) { return give(p, true); }
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamCreate(hipStream_t* s) { return *s = (hipStream_t)1, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = (hipEvent_t)1, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return busy ? result(hipErrorNotReady) : hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) {
    EXPECT(holds(p, n));
    if (holds(p, n)) memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { return hipMemset(p, v, n); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind kind) {
    const bool ok = (kind == hipMemcpyDeviceToHost || holds(d, n)) &&
                    (kind == hipMemcpyHostToDevice || holds(s, n));
    EXPECT(ok);
    if (ok) memmove(d, s, n);
    copies += kind == hipMemcpyDeviceToHost;
    return ok ? hipSuccess : result(hipErrorInvalidValue);
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind kind, hipStream_t) {
    return hipMemcpy(d, s, n, kind);
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
    const auto* b = find(p);
    if (!b) return result(hipErrorInvalidValue);
    memset(a, 0, sizeof(*a));
    a->type = b->second.host ? hipMemoryTypeHost : hipMemoryTypeDevice;
    a->devicePointer = const_cast<void*>(p);
    return hipSuccess;
}
hipError_t hipMemGetAddressRange(hipDeviceptr_t* base, size_t* size, hipDeviceptr_t p) {
    const auto* b = find(p);
    if (!b) return result(hipErrorInvalidValue);
    *base = b->first;
    *size = b->second.bytes;
    return hipSuccess;
}
}  // extern "C"

/* ---- the kernel launches ------------------------------------------------------ */
namespace lbmk {
int readout_blocks(int Nx, int Ny) { return ((Nx + 63) / 64) * ((Ny + 7) / 8); }

hipError_t launch_moments_f32(const Grid& g, const Phys&, const float* f, const float*, const float* T,
                              const Moments& out, int64_t, const unsigned long long* stat,
                              const Readout& ro, hipStream_t) {
    const size_t bytes = (size_t)g.Nx * g.Ny * sizeof(double);
    const int nb = readout_blocks(g.Nx, g.Ny);
    const bool ok = holds(f, 9 * (size_t)g.plane * 4) && holds(T, (size_t)g.plane * 4) &&
                    holds(stat, kStepWords * 8) && holds(ro.words, kStepWords * 8) &&
                    holds(ro.bad, nb * sizeof(unsigned));
    EXPECT(ok);
    if (!ok) return hipGetLastError();
    told = out;
    double* const to[4] = {out.rho, out.ux, out.uy, out.T};
    for (int q = 0; q < 4; ++q) {
        if (!to[q]) continue;
        EXPECT(holds(to[q], bytes));
        if (holds(to[q], bytes))
            for (int i = 0; i < g.Nx * g.Ny; ++i) to[q][i] = 10.0 * g.Nx + q;
    }
    memcpy(ro.words, stat, kStepWords * 8);
    memset(ro.bad, 0, nb * sizeof(unsigned));
    return hipGetLastError();
}
hipError_t launch_init_f32(const Grid& g, const Phys&, const double* rho0, float* f, float*, float* T,
                           hipStream_t) {
    EXPECT(holds(rho0, (size_t)g.Nx * g.Ny * sizeof(double)));
    EXPECT(holds(f, 9 * (size_t)g.plane * 4) && holds(T, (size_t)g.plane * 4));
    return hipGetLastError();
}
hipError_t launch_step_batched(const Slot* slots, int n, int, int, int, bool, hipStream_t) {
    EXPECT(holds(slots, n * sizeof(Slot)));
    return hipGetLastError();
}
hipError_t launch_step_f32(const Grid&, const Phys&, const Bufs<float>& b, bool, int64_t, hipStream_t) {
    EXPECT(holds(b.base, b.span));
    return hipGetLastError();
}
/* not reached here */
hipError_t launch_init_f64(const Grid&, const Phys&, const double*, double*, double*, hipStream_t) { abort(); }
hipError_t launch_moments_f64(const Grid&, const Phys&, const double*, const double*, const Moments&, int64_t,
                              const unsigned long long*, const Readout&, hipStream_t) { abort(); }
hipError_t launch_step_f64(const Grid&, const Phys&, const Bufs<double>&, int64_t, hipStream_t) { abort(); }
hipError_t launch_reduce(const double*, const double*, const double*, const double*, int, double, double*,
                         double*, hipStream_t) { abort(); }
hipError_t launch_reduce_state_f32(const Grid&, const Phys&, const float*, const float*, const float*, double,
                                   int64_t, double*, hipStream_t) { abort(); }
hipError_t launch_reduce_state_f64(const Grid&, const Phys&, const double*, const double*, double, int64_t,
                                   double*, hipStream_t) { abort(); }
hipError_t launch_copy(const void* s, void* d, size_t n, hipStream_t) {
    EXPECT(holds(s, n) && holds(d, n));
    return hipGetLastError();
}
}  // namespace lbmk

/* ---- the checks ------------------------------------------------------------------ */
static lbm_params channel(int Nx, int Ny) {
    lbm_params p;
    lbm_params_default(&p);
    p.Nx = Nx;
    p.Ny = Ny;
    EXPECT(lbm_params_resolve(&p) == LBM_OK);
    return p;
}

static void read_out(lbm_pool* P, int slot, const lbm_params& p) {
    std::vector<double> a[4];
    for (auto& v : a) v.assign((size_t)p.Nx * p.Ny, -1.0);
    EXPECT(lbm_pool_moments(P, slot, a[0].data(), a[1].data(), a[2].data(), a[3].data()) == LBM_OK);
    for (int q = 0; q < 4; ++q) EXPECT(a[q].front() == 10.0 * p.Nx + q && a[q].back() == 10.0 * p.Nx + q);
}

/* A small slot lives while a larger one is admitted and the k-th allocation
 * of that admission fails: the admission reports it, and the small slot, a
 * second larger one and one in between are read out as if nothing had been. */
static bool admission(int k) {
    where = "admission " + std::to_string(k);
    const lbm_params small = channel(64, 20), large = channel(300, 90), mid = channel(130, 60);
    lbm_pool* P = nullptr;
    int32_t a = -1, b = -1, c = -1;
    EXPECT(lbm_pool_create((size_t)1 << 30, nullptr, &P) == LBM_OK);
    EXPECT(lbm_pool_admit(P, &small, nullptr, 10, &a) == LBM_OK);
    fail_at = allocs + k;
    const lbm_status st = lbm_pool_admit(P, &large, nullptr, 10, &b);
    const bool failed = allocs > fail_at;
    fail_at = -1;
    EXPECT(failed || st == LBM_OK);
    read_out(P, a, small);
    EXPECT(lbm_pool_admit(P, &mid, nullptr, 10, &c) == LBM_OK);
    read_out(P, c, mid);
    if (b >= 0) read_out(P, b, large);
    EXPECT(lbm_pool_admit(P, &large, nullptr, 10, &b) == LBM_OK);
    read_out(P, b, large);
    EXPECT(lbm_pool_run(P, 10) == LBM_OK);
    read_out(P, a, small);
    EXPECT(lbm_pool_destroy(P) == LBM_OK);
    EXPECT(blocks.empty());
    return failed;
}

/* The same for a pool's first admission. */
static bool first(int k) {
    where = "first " + std::to_string(k);
    const lbm_params p = channel(64, 20);
    lbm_pool* P = nullptr;
    int32_t a = -1;
    EXPECT(lbm_pool_create((size_t)1 << 30, nullptr, &P) == LBM_OK);
    fail_at = allocs + k;
    const lbm_status st = lbm_pool_admit(P, &p, nullptr, 10, &a);
    const bool failed = allocs > fail_at;
    fail_at = -1;
    EXPECT((st != LBM_OK) == failed && (a < 0) == failed);
    if (failed) EXPECT(lbm_pool_admit(P, &p, nullptr, 10, &a) == LBM_OK);
    EXPECT(lbm_pool_run(P, 10) == LBM_OK);
    read_out(P, a, p);
    EXPECT(lbm_pool_destroy(P) == LBM_OK);
    EXPECT(blocks.empty());
    return failed;
}

/* The same for the batch's table, which a run of more slots makes larger: a
 * run of fewer slots then goes on as before. */
static bool run_growth(int k) {
    where = "run " + std::to_string(k);
    const lbm_params p = channel(64, 20);
    lbm_pool* P = nullptr;
    int32_t id[3];
    EXPECT(lbm_pool_create((size_t)1 << 30, nullptr, &P) == LBM_OK);
    EXPECT(lbm_pool_admit(P, &p, nullptr, 100, &id[0]) == LBM_OK);
    EXPECT(lbm_pool_run(P, 10) == LBM_OK);
    for (int i = 1; i < 3; ++i) EXPECT(lbm_pool_admit(P, &p, nullptr, 100, &id[i]) == LBM_OK);
    fail_at = allocs + k;
    const lbm_status st = lbm_pool_run(P, 10);
    const bool failed = allocs > fail_at;
    fail_at = -1;
    EXPECT((st != LBM_OK) == failed);
    for (int i = 1; i < 3; ++i) EXPECT(lbm_pool_release(P, id[i]) == LBM_OK);
    EXPECT(lbm_pool_run(P, 10) == LBM_OK);
    EXPECT(lbm_pool_slot_time(P, id[0]) == (failed ? 20 : 30));
    read_out(P, id[0], p);
    EXPECT(lbm_pool_destroy(P) == LBM_OK);
    EXPECT(blocks.empty());
    return failed;
}

/* A channel's creation without memory. */
static bool create(int k) {
    where = "create " + std::to_string(k);
    const lbm_params p = channel(300, 90);
    lbm_sim* s = nullptr;
    fail_at = allocs + k;
    const lbm_status st = lbm_create(&p, nullptr, nullptr, 0, nullptr, &s);
    const bool failed = allocs > fail_at;
    fail_at = -1;
    EXPECT(st == (failed ? LBM_ENOMEM : LBM_OK) && (s == nullptr) == failed);
    EXPECT(lbm_destroy(s) == LBM_OK && blocks.empty());
    (void)hipGetLastError();
    return failed;
}

/* A channel while another's creation, its tuning or the bandwidth probe finds
 * no memory: its next step and read-out are not told of it. */
static bool channel_calls(int k) {
    where = "channel " + std::to_string(k);
    const lbm_params p = channel(64, 20), q = channel(300, 90);
    const auto failing = [&](auto call) {
        lbm_sim* s = nullptr;
        EXPECT(lbm_create(&p, nullptr, nullptr, 0, nullptr, &s) == LBM_OK);
        fail_at = allocs + k;
        const lbm_status st = call(s);
        const bool failed = allocs > fail_at;
        fail_at = -1;
        EXPECT((st != LBM_OK) == failed);
        EXPECT(lbm_step(s, 2) == LBM_OK);
        std::vector<double> T((size_t)p.Nx * p.Ny);
        EXPECT(lbm_moments(s, nullptr, nullptr, nullptr, T.data()) == LBM_OK && T.back() == 10.0 * p.Nx + 3);
        EXPECT(lbm_destroy(s) == LBM_OK && blocks.empty());
        return failed;
    };
    bool any = failing([&](lbm_sim*) {
        lbm_sim* o = nullptr;
        const lbm_status st = lbm_create(&q, nullptr, nullptr, 0, nullptr, &o);
        EXPECT((o != nullptr) == (st == LBM_OK));
        EXPECT(lbm_destroy(o) == LBM_OK);
        return st;
    });
    any |= failing([](lbm_sim* s) { return lbm_autotune(s, 2, nullptr); });
    any |= failing([](lbm_sim*) { return lbm_bandwidth_probe(1 << 20, 2, nullptr, nullptr); });
    return any;
}

/* Freeing memory waits for the device, so an admission that the moment
 * arrays have room for frees nothing, though its read-out takes more
 * workgroups than any before (65 x 57 against 64 x 64 nodes). */
static bool growth(int k) {
    where = "growth";
    const lbm_params sizes[] = {channel(64, 64), channel(65, 57), channel(129, 30), channel(193, 21)};
    lbm_pool* P = nullptr;
    int32_t id[4];
    EXPECT(lbm_pool_create((size_t)1 << 30, nullptr, &P) == LBM_OK);
    for (int i = 0; i < 4; ++i) {
        const long before = frees;
        EXPECT(lbm_pool_admit(P, &sizes[i], nullptr, 10, &id[i]) == LBM_OK);
        EXPECT(frees == before);
    }
    for (int i = 0; i < 4; ++i) read_out(P, id[i], sizes[i]);
    EXPECT(lbm_pool_destroy(P) == LBM_OK);
    EXPECT(blocks.empty());
    return k < 1;
}

/* Who writes a read-out's pinned arrays: the kernel while no other slot's
 * steps run beside it and the arrays are within the line, a copy otherwise. */
static bool readout(int k) {
    where = "readout";
    const lbm_params p[2] = {channel(64, 20), channel(2048, 256)};  // the line: 16 MiB
    const lbm_params above = channel(2049, 256);
    lbm_pool* P = nullptr;
    int32_t id[2], big;
    EXPECT(lbm_pool_create((size_t)1 << 30, nullptr, &P) == LBM_OK);
    for (int i = 0; i < 2; ++i) EXPECT(lbm_pool_admit(P, &p[i], nullptr, i ? 20 : 10, &id[i]) == LBM_OK);
    EXPECT(lbm_pool_admit(P, &above, nullptr, 10, &big) == LBM_OK);
    const auto direct = [&](int slot, const lbm_params& q) {
        const size_t cells = (size_t)q.Nx * q.Ny;
        void* mem = nullptr;
        EXPECT(hipHostMalloc(&mem, 4 * cells * sizeof(double), 0) == hipSuccess);
        double* a = static_cast<double*>(mem);
        EXPECT(lbm_pool_moments(P, slot, a, a + cells, a + 2 * cells, a + 3 * cells) == LBM_OK);
        for (int f = 0; f < 4; ++f)
            EXPECT(a[f * cells] == 10.0 * q.Nx + f && a[(f + 1) * cells - 1] == 10.0 * q.Nx + f);
        const bool d = told.rho == a;
        EXPECT((told.ux == a + cells) == d && (told.T == a + 3 * cells) == d);
        EXPECT(hipHostFree(mem) == hipSuccess);
        return d;
    };
    EXPECT(lbm_pool_run(P, 10) == LBM_OK);
    busy = true;  // its own chunk is the last one: nothing runs after it
    EXPECT(direct(id[0], p[0]) && direct(id[1], p[1]) && !direct(big, above));
    EXPECT(lbm_pool_run(P, 10) == LBM_OK);  // the second slot alone
    EXPECT(!direct(id[0], p[0]) && direct(id[1], p[1]) && hipGetLastError() == hipSuccess);
    busy = false;
    EXPECT(direct(id[0], p[0]) && direct(id[1], p[1]));
    EXPECT(lbm_pool_destroy(P) == LBM_OK);
    // a channel's line, over the arrays that are asked for
    void* mem = nullptr;
    const size_t cells = ((size_t)4 << 20) / 32;
    EXPECT(hipHostMalloc(&mem, 8 * cells * sizeof(double), 0) == hipSuccess);
    double* a = static_cast<double*>(mem);
    double dev[4];
    double* const d[4] = {dev, dev + 1, dev + 2, dev + 3};
    double* const four[4] = {a, a + cells, a + 2 * cells, a + 3 * cells};
    double* const four1[4] = {a, a + cells + 1, a + 2 * cells + 2, a + 3 * cells + 3};
    double* const two[4] = {a, nullptr, a + 2 * cells, nullptr};
    const size_t line = lbmhost::kDirectChannel;
    EXPECT(lbmhost::plan_readout(four, d, cells, line).direct.rho == a);
    EXPECT(lbmhost::plan_readout(four1, d, cells + 1, line).direct.rho == dev);
    EXPECT(lbmhost::plan_readout(two, d, 2 * cells, line).direct.uy == a + 2 * cells);
    EXPECT(lbmhost::plan_readout(two, d, 2 * cells, line).direct.ux == nullptr);
    EXPECT(hipHostFree(mem) == hipSuccess);
    EXPECT(blocks.empty());
    return k < 1;
}

/* Copies of a read-out: one for arrays that follow one another in a pinned
 * allocation, one each where they do not, where the run of them leaves its
 * allocation for one that happens to adjoin, or in memory that is not pinned. */
static bool merge(int k) {
    where = "merge";
    const size_t cells = 1000, bytes = cells * sizeof(double);
    double* dev = nullptr;
    double* pin = nullptr;
    EXPECT(hipMalloc((void**)&dev, 4 * bytes) == hipSuccess && hipHostMalloc((void**)&pin, 5 * bytes, 0) == hipSuccess);
    for (size_t i = 0; i < 4 * cells; ++i) dev[i] = (double)i;
    double* const d[4] = {dev, dev + cells, dev + 2 * cells, dev + 3 * cells};
    const auto run = [&](double* a, double* b, double* c, double* e) {
        double* const to[4] = {a, b, c, e};
        memset(pin, 0, 5 * bytes);
        const int before = copies;
        EXPECT(lbmhost::enqueue_copies(lbmhost::plan_readout(to, d, cells, 0), cells, nullptr) == hipSuccess);
        for (int q = 0; q < 4; ++q)
            if (to[q]) EXPECT(memcmp(to[q], d[q], bytes) == 0);
        return copies - before;
    };
    double* const p = pin;
    EXPECT(run(p, p + cells, p + 2 * cells, p + 3 * cells) == 1);
    EXPECT(run(p, p + cells, p + 2 * cells + 1, p + 3 * cells + 1) == 2);
    EXPECT(run(p + cells, p, p + 3 * cells, p + 2 * cells) == 4);
    EXPECT(run(p, nullptr, p + 2 * cells, p + 3 * cells) == 2);
    EXPECT(run(nullptr, nullptr, nullptr, p) == 1 && run(nullptr, nullptr, nullptr, nullptr) == 0);
    std::vector<double> page(4 * cells);
    EXPECT(run(&page[0], &page[cells], &page[2 * cells], &page[3 * cells]) == 4);
    blocks[(char*)p].bytes = 2 * bytes;  // split into two that adjoin
    blocks[(char*)(p + 2 * cells)] = {3 * bytes, true};
    EXPECT(run(p, p + cells, p + 2 * cells, p + 3 * cells) == 3);  // two in the second
    blocks.erase((char*)(p + 2 * cells));
    EXPECT(hipHostFree(pin) == hipSuccess && hipFree(dev) == hipSuccess && blocks.empty());
    return k < 1;
}

/* The order of a step's tiles: every tile is taken by exactly one workgroup,
 * whatever the grid, alone on either kind of step and in a batch; a tile of a
 * batch meets the same XCD on every step, and each XCD takes its tiles on odd
 * steps in the reverse of the even ones' order. */
static lbmk::Grid grid(int Nx, int Ny, int seg_rows, bool in_batch) {
    const lbm_params p = channel(Nx, Ny);
    lbmhost::Layout L;
    lbmk::Grid g = {};
    EXPECT(lbmhost::make_layout(p, &L));
    lbmhost::fill_grid(p, L, seg_rows, lbmhost::tile_for(p, seg_rows), g, in_batch);
    EXPECT(g.n_blocks % 8 == 0);
    return g;
}
static bool order(int k) {
    where = "order";
    for (int strips = 1; strips <= 70; ++strips)
        for (int rows : {2, 14, 15, 100})
            for (int down = 0; down < 2; ++down) {
                const lbmk::Grid g = grid(54 * strips, rows + 2, 14, false);
                std::vector<int> taken(g.n_strips * g.n_segs, 0);
                int strip, seg;
                for (int b = 0; b < g.n_blocks; ++b)
                    if (lbmk::tile_of_block(g, b, b & 7, down, strip, seg)) ++taken[seg * g.n_strips + strip];
                for (int n : taken) EXPECT(n == 1);
            }
    const int sizes[][2] = {{64, 20}, {3000, 60}, {500, 100}, {55, 400}, {108, 31}};
    std::vector<lbmk::Grid> g;
    std::vector<int> begin;
    int total = 0, tiles = 0;
    for (auto& s : sizes) {
        g.push_back(grid(s[0], s[1], 14, true));
        begin.push_back(total);
        total += g.back().n_blocks;
        tiles += g.back().n_strips * g.back().n_segs;
    }
    std::vector<long> seen[2][8];  // tile numbers in the order an XCD takes them
    for (int step = 0; step < 2; ++step) {
        size_t n = 0;
        for (int wg = 0; wg < total; ++wg) {
            const int block = lbmk::batch_block(wg, total, step);
            size_t slot = 0;
            while (slot + 1 < g.size() && begin[slot + 1] <= block) ++slot;
            int strip, seg;
            if (!lbmk::tile_of_block(g[slot], block - begin[slot], wg & 7, false, strip, seg)) continue;
            seen[step][wg & 7].push_back((long)slot * 1000000 + seg * 1000 + strip);
            ++n;
        }
        EXPECT((int)n == tiles);
    }
    for (int x = 0; x < 8; ++x) {
        std::vector<long> back(seen[1][x].rbegin(), seen[1][x].rend());
        EXPECT(back == seen[0][x]);
    }
    return k < 1;
}

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "admission";
    int k = 0;
    while (k < 100 && (what == "first"     ? first(k)
                       : what == "run"     ? run_growth(k)
                       : what == "growth"  ? growth(k)
                       : what == "readout" ? readout(k)
                       : what == "create"  ? create(k)
                       : what == "channel" ? channel_calls(k)
                       : what == "merge"   ? merge(k)
                       : what == "order"   ? order(k)
                                           : admission(k)))
        ++k;
    printf("%s: %d turns, %d failed expectations\n", what.c_str(), k, failures);
    return failures || k == 0;
}
