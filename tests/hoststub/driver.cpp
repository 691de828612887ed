// The library's host code on the CPU (test tooling): this program defines
// the HIP runtime calls that libvpmc makes, so the host code runs with "device"
// memory from calloc, kernels that do nothing, allocations that fail and
// launches that are quicker where a case says so.  One case per run (argv[1]);
// each compares return codes and launches with the documented ones.  Exit
// status 0 when all agree.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/resource.h>
#include <time.h>

#include <map>
#include <vector>

#include "../../include/vpmc.h"

// ------------------------------------------------------------- HIP runtime
static const int kOutOfMemory = 2;
static std::map<void *, size_t> g_live;   // allocations
static size_t g_bytes = 0;                // their sum
static size_t g_room = ~(size_t)0;        // device memory: what does not fit is refused
static int g_last = 0;                    // what hipGetLastError has to say
static unsigned long long g_launches = 0, g_launches512 = 0;   // (those of 512 threads a workgroup)
static bool g_quick512 = false;                                // events take half the time around such launches
struct Dim3 {
    unsigned x, y, z;
};
static Dim3 g_grid, g_block;
static size_t g_shared;
static void *g_stream;

extern "C" {
int hipMalloc(void **p, size_t n) {
    if (n > g_room - (g_bytes < g_room ? g_bytes : g_room)) return g_last = kOutOfMemory;
    *p = calloc(1, n ? n : 1);
    g_live[*p] = n;
    g_bytes += n;
    return 0;
}
int hipFree(void *p) {
    auto it = g_live.find(p);
    if (it == g_live.end()) return g_last = 1;
    g_bytes -= it->second;
    g_live.erase(it);
    free(p);
    return 0;
}
int hipMemcpy(void *d, const void *s, size_t n, int) {
    if (n && (!d || !s)) return g_last = 1;
    if (n) memcpy(d, s, n);
    return 0;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *) { return hipMemcpy(d, s, n, k); }
int hipMemset(void *d, int v, size_t n) {
    if (n && !d) return g_last = 1;
    if (n) memset(d, v, n);
    return 0;
}
int hipMemsetAsync(void *d, int v, size_t n, void *) { return hipMemset(d, v, n); }
int hipLaunchKernel(const void *, Dim3 g, Dim3 b, void **, size_t, void *) {
    // the hardware's limit on a launch
    if ((unsigned long long)g.x * b.x >= 1ull << 32) return g_last = 9;
    ++g_launches;
    g_launches512 += b.x == 512;
    return 0;
}
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t shared, void *stream) {
    g_grid = g;
    g_block = b;
    g_shared = shared;
    g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *shared, void **stream) {
    *g = g_grid;
    *b = g_block;
    *shared = g_shared;
    *stream = g_stream;
    return 0;
}
int hipGetLastError() {
    const int e = g_last;
    g_last = 0;
    return e;
}
const char *hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : "error"; }
int hipGetDevice(int *d) { return *d = 0; }
int hipGetDeviceCount(int *n) { return *n = 1, 0; }
int hipSetDevice(int) { return 0; }
int hipGetDevicePropertiesR0600(void *, int) { return 1; }   // (the library then takes its defaults)
int hipMemGetInfo(size_t *f, size_t *t) { return *f = *t = (size_t)1 << 30, 0; }
int hipGetSymbolAddress(void **p, const void *) {
    static void *scratch = calloc(1, (size_t)32 << 20);
    return *p = scratch, 0;
}
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { return *s = malloc(1), 0; }
int hipStreamDestroy(void *s) { return free(s), 0; }
int hipEventCreate(void **e) { return *e = calloc(1, sizeof g_launches512), 0; }
int hipEventDestroy(void *e) { return free(e), 0; }
int hipEventRecord(void *e, void *) { return *(unsigned long long *)e = g_launches512, 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) {
    *ms = g_quick512 && *(unsigned long long *)a != *(unsigned long long *)b ? 0.5f : 1.0f;
    return 0;
}
}

// ------------------------------------------------------------- cases
static int fails = 0;
#define EXPECT(call, code)                                                                       \
    do {                                                                                         \
        const int rc_ = (call);                                                                  \
        if (rc_ != (code)) {                                                                     \
            fprintf(stderr, "line %d: %s returned %d, expected %d (%s)\n", __LINE__, #call, rc_, \
                    (code), vpmc_last_error(nullptr));                                           \
            fails++;                                                                             \
        }                                                                                        \
    } while (0)

static const float kSp[3] = {2.0f, 2.0f, 2.0f}, kOrg[3] = {-32.0f, -32.0f, 0.0f};
static const vpmc_beam kBeam = {{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
static const vpmc_spot kSpots[2] = {{0, 0, 150.0f, 3.0f, 0.0f, 1.0f, 1000}, {2.5f, 0, 140.0f, 3.0f, 0.0f, 1.0f, 500}};
static const vpmc_scenario kScen = {{0, 0, 0}, 1.0f};

static int load(vpmc_ctx *c, int n) {
    std::vector<int16_t> hu((size_t)n * n * n, 0);
    return vpmc_load_geometry(c, VPMC_GEOM_HU, hu.data(), n, n, n, kSp, kOrg, 0);
}

static int dense(vpmc_ctx *c, int n, size_t cap = 0, int batches = 0, int blocks = 0) {
    std::vector<float> dose((size_t)n * n * n);
    vpmc_opts o{};
    o.physics = VPMC_PHYS_ALL;
    o.max_device_bytes = cap;
    o.n_batches = batches;
    o.grid_blocks = blocks;
    return vpmc_run_spots(c, 0, kSpots, 2, &kScen, 1, &o, dose.data(), nullptr, nullptr, nullptr);
}

// a CT grid whose density array does not fit: the context has no geometry
// until one loads, and no run reads what the failed call released
static void geometry(vpmc_ctx *c) {
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    EXPECT(load(c, 8), VPMC_OK);
    EXPECT(dense(c, 8), VPMC_OK);
    g_room = g_bytes + 80000;   // 32^3: CT numbers of 66 kB fit, densities of 139 kB do not
    EXPECT(load(c, 32), VPMC_E_OOM);
    g_room = ~(size_t)0;
    EXPECT(dense(c, 8), VPMC_E_STATE);
    EXPECT(load(c, 32), VPMC_OK);
    EXPECT(dense(c, 32), VPMC_OK);
}

static std::vector<float> circle(int n, float r) {
    std::vector<float> p(2 * n);
    for (int i = 0; i < n; ++i) {
        p[2 * i] = r * cosf(6.2831853f * (i + 0.5f) / n);
        p[2 * i + 1] = r * sinf(6.2831853f * (i + 0.5f) / n);
    }
    return p;
}

// an opening whose raster does not fit: the field is not set until a call
// succeeds, and no run reads the polygon or raster that the failed call released
static void aperture(vpmc_ctx *c) {
    const vpmc_block blk = {30.0f, 8.5f, 50.0f};
    const std::vector<float> small = circle(16, 5.0f), large = circle(1000, 90.0f);
    EXPECT(load(c, 8), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, small.data(), 16, &blk, nullptr), VPMC_OK);
    EXPECT(dense(c, 8), VPMC_OK);
    g_room = g_bytes + 20000;
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, large.data(), 1000, &blk, nullptr), VPMC_E_OOM);
    g_room = ~(size_t)0;
    EXPECT(dense(c, 8), VPMC_E_STATE);
    // what the argument checks refuse leaves the field as it is
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, large.data(), 1000, &blk, nullptr), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, large.data(), 2, &blk, nullptr), VPMC_E_POLYGON);
    EXPECT(dense(c, 8), VPMC_OK);
}

static int matrix(vpmc_ctx *c, int n_spots, int hist = 100) {
    std::vector<vpmc_spot> sp(n_spots, kSpots[0]);
    for (vpmc_spot &s : sp) s.n_histories = (uint32_t)hist;
    std::vector<int64_t> rp(n_spots + 1);
    vpmc_opts o{};
    o.physics = VPMC_PHYS_ALL;
    o.output = VPMC_OUT_CSR;
    return vpmc_run_spots(c, 0, sp.data(), n_spots, &kScen, 1, &o, nullptr, nullptr, nullptr, rp.data());
}

// more row slots than fit: the slots that were there are gone, and the next
// run allocates its own
static void slots(vpmc_ctx *c) {
    EXPECT(load(c, 8), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    EXPECT(matrix(c, 2), VPMC_OK);
    g_room = g_bytes + 100000;   // 60 slots of 4 KB do not fit
    EXPECT(matrix(c, 60), VPMC_E_OOM);
    g_room = ~(size_t)0;
    const size_t before = g_bytes;
    EXPECT(matrix(c, 2), VPMC_OK);
    if (g_bytes < before + 2 * 512 * 8) {
        fprintf(stderr, "the run after the failed one has no row slots\n");
        fails++;
    }
}

// a dense run whose batch grids and staging do not fit together: it runs batch
// by batch in the room that a run batch by batch needs
static void fallback(vpmc_ctx *c) {
    const size_t n = 32, nvox = n * n * n;
    EXPECT(load(c, (int)n), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    // tally, batch grid, squares, staged dose and small tables; the queue
    // wants 16 batch grids, or the staging of 1500 particles beside these
    g_room = g_bytes + nvox * (8 + 8 + 8 + 4) + 16384;
    EXPECT(dense(c, (int)n, 0, 16), VPMC_OK);
    g_room = ~(size_t)0;
    EXPECT(dense(c, (int)n, 0, 16), VPMC_OK);
}

// a call refused for memory does not fail the next one (launches report the
// runtime's last error)
static void next_call(vpmc_ctx *c) {
    EXPECT(load(c, 8), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    EXPECT(dense(c, 8), VPMC_OK);
    EXPECT(matrix(c, 2), VPMC_OK);
    g_room = g_bytes + 100000;
    EXPECT(matrix(c, 60), VPMC_E_OOM);
    EXPECT(dense(c, 8), VPMC_OK);
    EXPECT(load(c, 32), VPMC_E_OOM);
    EXPECT(load(c, 8), VPMC_OK);
    std::vector<float> w(vpmc_surrogate_param_count(), 0.01f), x(8 * 64, 0.1f), y(3 * 64, 0.1f), t(64, 1.0f);
    EXPECT(vpmc_surrogate_set_weights(c, w.data(), (int)w.size()), VPMC_E_OOM);
    g_room = ~(size_t)0;
    EXPECT(vpmc_surrogate_set_weights(c, w.data(), (int)w.size()), VPMC_OK);
    g_room = g_bytes + 100000;   // the fragments and partial gradients do not fit
    EXPECT(vpmc_surrogate_loss_grad(c, x.data(), y.data(), t.data(), 64, w.data(), nullptr), VPMC_E_OOM);
    g_room = ~(size_t)0;
    EXPECT(vpmc_surrogate_loss_grad(c, x.data(), y.data(), t.data(), 64, w.data(), nullptr), VPMC_OK);
}

static int noalloc(vpmc_ctx *c) {
    vpmc_opts o{};
    o.physics = VPMC_PHYS_ALL;
    o.flags = VPMC_DEVICE_PTRS;
    double led[VPMC_NLEDGER];
    return vpmc_run_spots_noalloc(c, 0, kSpots, 2, &kScen, 1, &o, nullptr, nullptr, led);
}

// Dense runs tuned through the work queue: the untuned default is a candidate
// (and wins where nothing is faster), smaller workgroups come as resident sets,
// and the pick does not shape the batch-by-batch kernel, which has its own.
static void autotune(vpmc_ctx *c) {
    EXPECT(load(c, 16), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    vpmc_opts base{}, best{};
    base.physics = VPMC_PHYS_ALL;
    auto tune = [&](int threads, int blocks) {
        EXPECT(vpmc_autotune(c, 0, kSpots, 2, &kScen, &base, 1000, &best), VPMC_OK);
        EXPECT(best.block_threads, threads);
        EXPECT(best.grid_blocks, blocks);
        EXPECT(dense(c, 16), VPMC_OK);
        std::vector<float> dose(16 * 16 * 16);
        EXPECT(vpmc_run_spots(c, 0, kSpots, 2, &kScen, 1, &best, dose.data(), nullptr, nullptr, nullptr), VPMC_OK);
    };
    tune(0, 0);
    g_quick512 = true;
    tune(512, 256 * 16 / 8);
    unsigned long long n = g_launches512;
    EXPECT(dense(c, 16, 0, 2), VPMC_OK);   // (with batches: through the queue at any size)
    EXPECT(g_launches512 > n, true);
    n = g_launches512;
    EXPECT(noalloc(c), VPMC_OK);
    EXPECT(dense(c, 16, (size_t)1 << 30), VPMC_OK);
    EXPECT(g_launches512 == n, true);
    g_quick512 = false;
    tune(0, 0);
    // the batch-by-batch route, by a cap on device memory
    g_quick512 = true;
    base.max_device_bytes = (size_t)1 << 30;
    tune(512, 4 * 256 * 256 / 512);
    n = g_launches512;
    EXPECT(noalloc(c), VPMC_OK);
    EXPECT(g_launches512 > n, true);
    n = g_launches512;
    EXPECT(dense(c, 16, 0, 2), VPMC_OK);
    EXPECT(g_launches512 == n, true);
}

// any grid_blocks that the argument checks accept: a dense run launches no more
// workgroups than run at once (what a launch can hold, with their staging)
static void blocks(vpmc_ctx *c) {
    EXPECT(load(c, 16), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    for (int b : {1, 37, 1 << 20, 1 << 24, 0x7fffffff}) EXPECT(dense(c, 16, 0, 0, b), VPMC_OK);
    for (int b : {1, 37, 1 << 20, 1 << 24, 0x7fffffff}) EXPECT(dense(c, 16, (size_t)1 << 30, 0, b), VPMC_OK);
}

// 1.1e12 histories in one dense run: the host's tables stay small
static void many_histories(vpmc_ctx *c) {
    EXPECT(load(c, 8), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    std::vector<vpmc_spot> sp(256, kSpots[0]);
    for (vpmc_spot &s : sp) s.n_histories = 0xffffffffu;
    std::vector<float> dose(8 * 8 * 8);
    vpmc_opts o{};
    o.physics = VPMC_PHYS_ALL;
    g_room = g_bytes + ((size_t)256 << 20);
    EXPECT(vpmc_run_spots(c, 0, sp.data(), 256, &kScen, 1, &o, dose.data(), nullptr, nullptr, nullptr), VPMC_OK);
    struct rusage u;
    getrusage(RUSAGE_SELF, &u);
    if (u.ru_maxrss > 1 << 20) {   // (kB)
        fprintf(stderr, "the run took %ld MB of host memory\n", u.ru_maxrss / 1024);
        fails++;
    }
}

// smallest max_device_bytes that lets a dense run through
static size_t least_cap(vpmc_ctx *c, int n) {
    for (size_t cap = (size_t)n * n * n * 8; cap < (size_t)64 << 20; cap += 256)
        if (dense(c, n, cap) == VPMC_OK) return cap;
    return 0;
}

// what max_device_bytes is held against does not drift with allocations that
// failed before
static void counted(vpmc_ctx *c) {
    const vpmc_block blk = {30.0f, 8.5f, 50.0f};
    const std::vector<float> small = circle(16, 30.0f), large = circle(1000, 90.0f);
    EXPECT(load(c, 8), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, small.data(), 16, &blk, nullptr), VPMC_OK);
    g_room = g_bytes + 1200000;   // the distances of the larger raster fit, its cells do not
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, large.data(), 1000, &blk, nullptr), VPMC_E_OOM);
    g_room = ~(size_t)0;
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, large.data(), 1000, &blk, nullptr), VPMC_OK);
    vpmc_ctx *d = nullptr;
    EXPECT(vpmc_create(&d, 0), VPMC_OK);
    EXPECT(load(d, 8), VPMC_OK);
    EXPECT(vpmc_set_aperture(d, 0, &kBeam, large.data(), 1000, &blk, nullptr), VPMC_OK);
    const size_t a = least_cap(c, 8), b = least_cap(d, 8);
    if (!a || a != b) {
        fprintf(stderr, "least cap %zu after a failed call, %zu without one\n", a, b);
        fails++;
    }
    vpmc_destroy(d);
}

// dense and matrix runs of every choice of batches, scenarios, outputs and
// processes, from no spots on (for the sanitizers)
static void outputs(vpmc_ctx *c) {
    const vpmc_block blk = {30.0f, 8.5f, 50.0f};
    const std::vector<float> poly = circle(16, 5.0f);
    EXPECT(load(c, 8), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, poly.data(), 16, &blk, nullptr), VPMC_OK);
    const std::vector<vpmc_scenario> sc(5, kScen);
    for (int n : {0, 1, 65})
        for (int batches : {0, 2, 16, 1024})
            for (int S : {5, 1})
                for (unsigned flags : {0u, (unsigned)VPMC_LET, (unsigned)VPMC_DEVICE_PTRS})
                    for (unsigned physics : {0u, (unsigned)VPMC_PHYS_ALL}) {
                        std::vector<vpmc_spot> sp(n, kSpots[0]);
                        for (int i = 0; i < n; ++i) {
                            sp[i].n_histories = (uint32_t)(i * 37 % 300);
                            sp[i].x_mm = i == 3 ? 1e30f : i * 7.0f - 200.0f;
                        }
                        std::vector<float> dose(512 * S), sigma(512 * S);
                        std::vector<double> led(VPMC_NLEDGER * S);
                        std::vector<int64_t> rp((size_t)n * S + 1);
                        vpmc_opts o{};
                        o.physics = physics;
                        o.n_batches = batches;
                        o.flags = flags;
                        EXPECT(vpmc_run_spots(c, 0, sp.data(), n, sc.data(), S, &o, dose.data(),
                                              batches ? sigma.data() : nullptr, led.data(), nullptr), VPMC_OK);
                        o.flags &= ~VPMC_LET;
                        o.n_batches = 0;
                        o.output = VPMC_OUT_CSR;
                        o.max_slots = batches ? 3 : 0;
                        EXPECT(vpmc_run_spots(c, 0, sp.data(), n, sc.data(), S, &o, nullptr, nullptr, led.data(),
                                              rp.data()), VPMC_OK);
                    }
}

// a dense run of few histories is one transport and one conversion; with
// batches, or a launch shape that is asked for, it goes through the queue (beam
// line, boxes, queue, fold or conversion)
static void few(vpmc_ctx *c) {
    EXPECT(load(c, 16), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    auto launches = [&](int batches, int blocks) {
        const unsigned long long n = g_launches;
        EXPECT(dense(c, 16, 0, batches, blocks), VPMC_OK);
        return (int)(g_launches - n);
    };
    EXPECT(launches(0, 0), 2);
    EXPECT(launches(2, 0), 4);
    EXPECT(launches(0, 8), 4);
}

// 2e5 spots: what the host does for a run through the queue stays within six
// times what it does batch by batch (the quickest of three calls each)
static void many_spots(vpmc_ctx *c) {
    EXPECT(load(c, 8), VPMC_OK);
    EXPECT(vpmc_set_aperture(c, 0, &kBeam, nullptr, 0, nullptr, nullptr), VPMC_OK);
    std::vector<vpmc_spot> sp(200000, kSpots[0]);
    unsigned r = 1;
    auto rnd = [&]() { return (float)((r = r * 1664525u + 1013904223u) >> 8) / (1 << 24); };
    for (vpmc_spot &s : sp) {
        s.x_mm = 150.0f * rnd();
        s.y_mm = 150.0f * rnd();
        s.energy_mev = 70.0f + 150.0f * rnd();
        s.n_histories = 5;
    }
    std::vector<float> dose(512);
    double ms[2] = {1e30, 1e30};
    for (int pass = 0; pass < 6; ++pass) {
        vpmc_opts o{};
        o.physics = VPMC_PHYS_ALL;
        const int queue = pass / 3;
        o.max_device_bytes = queue ? 0 : (size_t)1 << 30;
        timespec a, b;
        clock_gettime(CLOCK_MONOTONIC, &a);
        EXPECT(vpmc_run_spots(c, 0, sp.data(), (int)sp.size(), &kScen, 1, &o, dose.data(), nullptr, nullptr, nullptr),
               VPMC_OK);
        clock_gettime(CLOCK_MONOTONIC, &b);
        ms[queue] = fmin(ms[queue], (b.tv_sec - a.tv_sec) * 1e3 + (b.tv_nsec - a.tv_nsec) * 1e-6);
    }
    printf("host time batch by batch %.2f ms, queue %.2f ms\n", ms[0], ms[1]);
    EXPECT(ms[1] <= 6.0 * ms[0], true);
}

int main(int argc, char **argv) {
    vpmc_ctx *c = nullptr;
    EXPECT(vpmc_create(&c, 0), VPMC_OK);
    const char *name = argc > 1 ? argv[1] : "";
    if (!strcmp(name, "geometry")) geometry(c);
    else if (!strcmp(name, "aperture")) aperture(c);
    else if (!strcmp(name, "slots")) slots(c);
    else if (!strcmp(name, "fallback")) fallback(c);
    else if (!strcmp(name, "next_call")) next_call(c);
    else if (!strcmp(name, "autotune")) autotune(c);
    else if (!strcmp(name, "blocks")) blocks(c);
    else if (!strcmp(name, "many_histories")) many_histories(c);
    else if (!strcmp(name, "counted")) counted(c);
    else if (!strcmp(name, "outputs")) outputs(c);
    else if (!strcmp(name, "few")) few(c);
    else if (!strcmp(name, "many_spots")) many_spots(c);
    else return 2;
    vpmc_destroy(c);
    if (!g_live.empty()) {
        fprintf(stderr, "%zu allocations left\n", g_live.size());
        fails++;
    }
    if (fails) return 1;
    printf("%s: ok\n", name);
    return 0;
}
