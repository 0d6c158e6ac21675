// The host path of libcubestats.so on a machine without a GPU: this program
// defines the HIP calls that the library makes (an executable's symbols come
// before those of the libraries it loads).  Device memory is host memory that
// nobody touches, kernels do not run, and every launch is noted in the order
// in which it was made.  Each scenario below drives entry points and exits 0,
// or prints what was wrong.
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <functional>
#include <map>
#include <mutex>
#include <string>
#include <thread>
#include <vector>

#include "cube_internal.h"

using cube::PassArgs;

#define CHECK(c)                                                  \
    do {                                                          \
        if (!(c)) {                                               \
            printf("%s:%d: %s\n", __FILE__, __LINE__, #c);        \
            printf("%s\n", cube_last_error());                    \
            dump_launches();                                      \
            exit(1);                                              \
        }                                                         \
    } while (0)

// ------------------------------------------------------------- the fake runtime
struct Launch {
    std::string name;
    dim3 grid;
    hipStream_t stream;
    std::thread::id thread;
    bool is_pass;     // `pass` holds the kernel's arguments
    PassArgs pass;
};

static std::mutex g_m;
// The library registers its kernels before this program's own objects exist.
static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> n;
    return n;
}
static std::map<uintptr_t, size_t> g_mem;      // device and pinned allocations
static std::vector<Launch> g_launches;
static std::map<uintptr_t, size_t> g_pinned;   // those in host memory
static std::vector<size_t> g_mallocs;          // sizes of device allocations, in order
static std::vector<uintptr_t> g_frees;
static std::function<void(const Launch &)> g_hook;  // after a launch was noted
static bool g_signal = true;                   // passes tell the host that they are done
static std::atomic<bool> g_capturing{false}, g_no_memory{false};
static thread_local struct { dim3 grid, block; size_t lds; hipStream_t s; } g_cfg;

static void dump_launches()
{
    for (const Launch &l : g_launches)
        printf("  stream %p thread %zx %s\n", (void *)l.stream,
               std::hash<std::thread::id>()(l.thread) & 0xffff, l.name.c_str());
    fflush(stdout);
}

static void *take(size_t n)
{
    n = (n + 4095) & ~(size_t)4095;
    void *p = mmap(nullptr, n, PROT_READ | PROT_WRITE,
                   MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED) abort();
    std::lock_guard<std::mutex> lk(g_m);
    g_mem[(uintptr_t)p] = n;
    return p;
}
static void give(void *p)
{
    if (!p) return;
    std::lock_guard<std::mutex> lk(g_m);
    auto it = g_mem.find((uintptr_t)p);
    if (it == g_mem.end()) abort();
    munmap(p, it->second);
    g_mem.erase(it);
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *x; return &x; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *,
                           void *, dim3 *, dim3 *, int *)
{
    names()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    g_cfg = {g, b, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    *g = g_cfg.grid;
    *b = g_cfg.block;
    *lds = g_cfg.lds;
    *s = g_cfg.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3, void **args, size_t, hipStream_t s)
{
    Launch l = {names().at(f), g, s, std::this_thread::get_id(), false, {}};
    l.is_pass = l.name.find("6k_passI") != std::string::npos ||
                l.name.find("10k_pass_dynI") != std::string::npos;
    if (l.is_pass) l.pass = *(const PassArgs *)args[0];
    {
        std::lock_guard<std::mutex> lk(g_m);
        g_launches.push_back(l);
    }
    if (g_hook) g_hook(l);
    if (l.is_pass && l.pass.done && g_signal)
        __atomic_store_n(l.pass.done, l.pass.done_gen, __ATOMIC_RELEASE);
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n)
{
    if (g_capturing) return hipErrorStreamCaptureUnsupported;
    if (g_no_memory) return hipErrorOutOfMemory;
    {
        std::lock_guard<std::mutex> lk(g_m);
        g_mallocs.push_back(n);
    }
    *p = take(n);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (p) {
        std::lock_guard<std::mutex> lk(g_m);
        g_frees.push_back((uintptr_t)p);
    }
    give(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned)
{
    *p = take(n);
    std::lock_guard<std::mutex> lk(g_m);
    g_pinned[(uintptr_t)*p] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void *p) { give(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t p)
{
    std::lock_guard<std::mutex> lk(g_m);
    auto it = g_mem.upper_bound((uintptr_t)p);
    if (it == g_mem.begin()) return hipErrorInvalidValue;
    --it;
    *base = (hipDeviceptr_t)it->first;
    *size = it->second;
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *)
{
    memset(a, 0, sizeof *a);
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t)
{
    return g_capturing ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st)
{
    *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "an error"; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)1; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
}

// ------------------------------------------------------------------ scenarios
static hipStream_t const STREAM = (hipStream_t)0x1000;

static float *device_floats(size_t n) { return (float *)take(n * 4); }

// Thread B makes its call while thread A is between two launches of its own;
// the launches of each call must still follow each other.
static void interleave(std::function<void()> a, std::function<void()> b)
{
    std::atomic<bool> started{false}, b_done{false};
    std::thread::id a_id = std::this_thread::get_id();
    g_launches.clear();
    g_hook = [&](const Launch &l) {
        if (l.thread != a_id || started.exchange(true)) return;
        const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(300);
        std::thread(
            [&] {
                b();
                b_done = true;
            })
            .detach();
        while (!b_done && std::chrono::steady_clock::now() < until) std::this_thread::yield();
    };
    a();
    while (!b_done) std::this_thread::yield();
    g_hook = nullptr;
    int changes = 0;
    for (size_t i = 1; i < g_launches.size(); ++i)
        changes += g_launches[i].thread != g_launches[i - 1].thread;
    CHECK(started && g_launches.size() >= 4 && changes == 1);
}

static void shared_stream()
{
    const int64_t n = 1 << 21, dims[5] = {n, 1, 1, 0, 0};
    float *x = device_floats(n), *y = device_floats(n);
    cube_stats_t *out = (cube_stats_t *)take(sizeof *out);
    uint64_t *c = (uint64_t *)take((65536 + 3) * 8);
    auto ok = [](int rc) {
        if (rc) printf("error: %s\n", cube_last_error());
        if (rc) exit(1);
    };
    for (int bins : {8192, 16384, 65536}) {
        auto fused = [&](float *p, hipStream_t s) {
            return [=] { ok(cube_stats_hist_async(p, dims, -1.f, 1.f, bins, out, c, s)); };
        };
        ok(cube_stats_hist_async(x, dims, -1.f, 1.f, bins, out, c, STREAM));
        interleave(fused(x, STREAM), fused(y, STREAM));
        // A synchronous call and a stream-ordered one on the default stream.
        std::vector<uint64_t> host((size_t)bins + 3);
        auto sync = [&] { ok(cube_hist(x, dims, -1.f, 1.f, bins, host.data())); };
        interleave(sync, fused(y, nullptr));
        interleave(fused(y, nullptr), sync);
    }
    auto minmax = [&](float *p) {
        return [=] { ok(cube_stats_hist_minmax_async(p, dims, 64, out, c, STREAM)); };
    };
    interleave(minmax(x), minmax(y));
}

static bool launched(const char *what)
{
    for (const Launch &l : g_launches)
        if (l.name.find(what) != std::string::npos) return true;
    return false;
}

static bool pinned(const void *p)
{
    auto it = g_pinned.upper_bound((uintptr_t)p);
    return it != g_pinned.begin() && (uintptr_t)p < (--it)->first + it->second;
}

// Whatever a synchronous call's passes leave in host memory is written through,
// by the pass that says that it is done; a min/max call's first pass leaves its
// statistics on the device for the second.
static void host_results()
{
    const int64_t n = 1 << 21, dims[5] = {n, 1, 1, 0, 0};
    float *x = device_floats(n);
    cube_stats_t st;
    std::vector<uint64_t> c(65536 + 3);
    int results = 0, forwarded = 0;
    for (int bins : {64, 8191, 8192, 65536}) {
        g_launches.clear();
        CHECK(cube_stats(x, n, 1, 1, nullptr, &st) == CUBE_OK);
        CHECK(cube_hist(x, dims, -1.f, 1.f, bins, c.data()) == CUBE_OK);
        CHECK(cube_stats_hist(x, dims, -1.f, 1.f, bins, &st, c.data()) == CUBE_OK);
        CHECK(cube_stats_hist_minmax(x, dims, bins, &st, c.data()) == CUBE_OK);
        const PassArgs *first = nullptr;
        for (const Launch &l : g_launches) {
            if (!l.is_pass) continue;
            const bool host = pinned(l.pass.out) || pinned(l.pass.counts);
            CHECK(host == (l.pass.host != 0) && (host || !l.pass.done));
            CHECK(!l.pass.done || pinned(l.pass.done));
            if (first) {
                CHECK(l.pass.stats_in == first->out && pinned(l.pass.out));
                ++forwarded;
            } else {
                CHECK(!l.pass.stats_in);
            }
            first = host ? nullptr : &l.pass;
            results += host;
        }
        CHECK(!first);
        // Stream-ordered: device memory, nothing forwarded.
        g_launches.clear();
        cube_stats_t *d_out = (cube_stats_t *)take(sizeof st);
        uint64_t *d_c = (uint64_t *)take((bins + 3) * 8);
        CHECK(cube_stats_hist_minmax_async(x, dims, bins, d_out, d_c, nullptr) == CUBE_OK);
        for (const Launch &l : g_launches)
            CHECK(!l.is_pass || (!l.pass.host && !l.pass.done && !l.pass.stats_in));
    }
    CHECK(results == 4 * 4 && forwarded == 4);
}

// A stream that completes without the pass's word: an error, not the results
// of the call before.
static void lost_results()
{
    const int64_t n = 1 << 20, dims[5] = {n, 1, 1, 0, 0};
    float *x = device_floats(n);
    cube_stats_t st;
    std::vector<uint64_t> c(64 + 3);
    double median;
    CHECK(cube_stats_hist(x, dims, -1.f, 1.f, 64, &st, c.data()) == CUBE_OK);
    g_signal = false;
    CHECK(cube_stats(x, n, 1, 1, nullptr, &st) == CUBE_EDEVICE);
    CHECK(cube_hist(x, dims, -1.f, 1.f, 64, c.data()) == CUBE_EDEVICE);
    CHECK(cube_stats_hist(x, dims, -1.f, 1.f, 64, &st, c.data()) == CUBE_EDEVICE);
    CHECK(cube_stats_hist_minmax(x, dims, 64, &st, c.data()) == CUBE_EDEVICE);
    CHECK(cube_median(x, dims, &median, nullptr) == CUBE_EDEVICE);
    g_signal = true;
    CHECK(cube_stats_hist(x, dims, -1.f, 1.f, 64, &st, c.data()) == CUBE_OK);
}

// Two threads project on one stream: each call's slices and the launch that
// merges them share the stream's partials, which the larger call also grows.
static void shared_projection()
{
    const int64_t small[5] = {64, 64, 256, 0, 0}, large[5] = {256, 256, 256, 0, 0};
    float *x = device_floats((size_t)256 * 256 * 256);
    float *mip = device_floats(256 * 256);
    auto project = [&](const int64_t *dims) {
        return [=] { CHECK(cube_project(x, dims, mip, nullptr, nullptr, STREAM) == CUBE_OK); };
    };
    interleave(project(large), project(large));
    interleave(project(small), project(large));
    cube_shutdown();
    interleave(project(small), project(large));  // the buffer grows in between
}

// A projection that would take slices makes do with one where their partials
// cannot be had: under capture, where nothing may be allocated or waited for,
// and without memory.
static void projection_without_partials()
{
    const int64_t dims[5] = {256, 256, 256, 0, 0}, more[5] = {517, 500, 256, 0, 0};
    float *x = device_floats((size_t)512 * 512 * 256);
    float *mip = device_floats(512 * 512);
    auto project = [&](const int64_t *d) {
        g_launches.clear();
        return cube_project(x, d, mip, nullptr, nullptr, STREAM);
    };
    for (int k = 0; k < 2; ++k) {
        std::atomic<bool> &no = k ? g_no_memory : g_capturing;
        no = true;
        CHECK(project(dims) == CUBE_OK && g_launches.size() == 1 && g_launches[0].grid.y == 1);
        no = false;
        CHECK(project(dims) == CUBE_OK && g_launches.size() == 2 && g_launches[0].grid.y > 1 &&
              launched("k_project_merge"));
        // The partials of an earlier call serve, too few of them do not.
        no = true;
        CHECK(project(dims) == CUBE_OK && g_launches.size() == 2);
        CHECK(project(more) == CUBE_OK && g_launches.size() == 1 && g_launches[0].grid.y == 1);
        no = false;
        CHECK(project(more) == CUBE_OK && g_launches.size() == 2);
        cube_shutdown();
    }
}

// A captured graph keeps the address of the partials: making room for more
// must not free them before cube_shutdown does.
static void captured_partials()
{
    const int64_t dims[5] = {256, 256, 256, 0, 0}, more[5] = {517, 500, 256, 0, 0};
    float *x = device_floats((size_t)517 * 500 * 256);
    float *mip = device_floats(517 * 500);
    auto project = [&](const int64_t *d) {
        CHECK(cube_project(x, d, mip, nullptr, nullptr, STREAM) == CUBE_OK);
    };
    project(dims);
    project(more);
    CHECK(g_frees.size() == 1);   // nothing was captured
    cube_shutdown();
    g_frees.clear();
    project(dims);
    g_capturing = true;
    project(dims);
    g_capturing = false;
    project(more);
    CHECK(g_frees.empty());
    cube_shutdown();
    CHECK(g_frees.size() == 2);
    project(dims);
}

// Which images take quads of pixels: whole ones of any size (their wavefronts
// count from their own first quad), others while a wavefront's offsets from
// its first row fit 32 bits.
static void projection_kernels()
{
    const int64_t K = 1024;
    struct { int64_t dims[5]; bool quads; } cases[] = {
        {{64 * K, 8 * K, 2, 0, 0}, true},                     // 2^29 pixels, dense
        {{64 * K, 32 * K + 1, 2, 0, 0}, true},                // over 2^31
        {{(int64_t)1 << 31, 1, 1, 0, 0}, true},
        {{4 * K, 4 * K, 2, (int64_t)1 << 28, (int64_t)1 << 40}, true},
        {{4 * K, 4 * K, 2, (int64_t)1 << 29, (int64_t)1 << 41}, false},
        {{3, 4 * K, 2, 4, 0}, false},
        {{3, 4 * K, 2 * K, 3, 0}, true}};                     // one row of 12 K pixels
    for (auto &c : cases) {
        const size_t npix = (size_t)(c.dims[0] * c.dims[1]);
        const int64_t *d = c.dims;
        const int64_t sy = d[3] ? d[3] : d[0], sz = d[4] ? d[4] : sy * d[1];
        const size_t end = (size_t)((d[2] - 1) * sz + (d[1] - 1) * sy + d[0]);
        float *x = device_floats(end), *mip = device_floats(npix);
        g_launches.clear();
        CHECK(cube_project(x, d, mip, nullptr, nullptr, STREAM) == CUBE_OK);
        CHECK(launched("k_project_quads") == c.quads && launched("9k_projectE") != c.quads);
        give(x);
        give(mip);
    }
}

// The kernel and the number of slices on 256 CUs, on both sides of each line.
static void projection_slices()
{
    struct { int64_t nx, ny, nz; bool quads; unsigned slices; } cases[] = {
        {64, 64, 16, false, 1},   {64, 64, 39, false, 1},    {64, 64, 40, false, 2},
        {64, 64, 512, false, 16}, {64, 64, 4608, false, 64}, {64, 64, 4609, true, 64},
        {256, 256, 288, false, 4}, {256, 256, 289, true, 6}, {450, 450, 93, false, 1},
        {450, 450, 94, true, 1},  {450, 450, 96, true, 2},   {512, 512, 72, false, 1},
        {512, 512, 73, true, 1},  {512, 512, 96, true, 2},   {550, 550, 256, false, 1},
        {550, 550, 257, true, 1}, {550, 550, 400, true, 2},  {600, 600, 399, true, 1},
        {600, 600, 400, true, 2}, {640, 640, 512, true, 1},  {640, 640, 16, false, 1},
        {640, 640, 17, true, 1},  {941, 937, 21, false, 1},  {941, 937, 22, true, 1},
        {4096, 4096, 1, false, 1}, {4096, 4096, 2, true, 1}};
    float *x = device_floats((size_t)1 << 28), *mip = device_floats((size_t)1 << 24);
    for (auto &c : cases) {
        const int64_t dims[5] = {c.nx, c.ny, c.nz, 0, 0};
        g_launches.clear();
        CHECK(cube_project(x, dims, mip, nullptr, nullptr, STREAM) == CUBE_OK);
        if (launched("k_project_quads") != c.quads || g_launches[0].grid.y != c.slices) {
            printf("%ld x %ld x %ld: %s, %u slices\n", (long)c.nx, (long)c.ny, (long)c.nz,
                   g_launches[0].name.c_str(), g_launches[0].grid.y);
            exit(1);
        }
    }
}

// A box of rows under four voxels (a pixel's spectrum) is visited row by row:
// every pass spreads its rows over the chip.
static void thin_rows()
{
    struct { int64_t nx, ny, nz; } cases[] = {{1, 1, 1000}, {1, 5, 1024}, {2, 200, 200},
                                              {3, 64, 1000}, {1, 1, 7},    {3, 1, 20000000}};
    float *x = device_floats((size_t)1 << 32);
    g_signal = false;    // no kernel runs: the calls end in an error
    for (auto &c : cases) {
        const int64_t dims[5] = {c.nx, c.ny, c.nz, 8, 8 * (c.ny + 1)};
        const double q[3] = {0.1, 0.5, 0.9};
        double v[3];
        float f;
        const unsigned want = (unsigned)std::min<int64_t>(512, c.ny * c.nz);
        cube_stats_t st;
        std::vector<uint64_t> counts(1024 + 3);
        for (int op = 0; op < 5; ++op) {
            g_launches.clear();
            if (op == 3) cube_stats_hist(x, dims, -1.f, 1.f, 1024, &st, counts.data());
            if (op == 4) cube_stats_hist_minmax(x, dims, 64, &st, counts.data());
            if (op == 0) cube_median(x, dims, v, nullptr);
            if (op == 1) cube_select(x, dims, 3, &f);
            if (op == 2) cube_quantiles(x, dims, q, 3, v, nullptr);
            bool seen = false;
            for (const Launch &l : g_launches) {
                const bool pass = l.is_pass || l.name.find("7k_quantI") != std::string::npos ||
                                  l.name.find("9k_bracketILi2E") != std::string::npos;
                if (pass) CHECK(l.grid.x >= want);
                seen |= pass;
            }
            CHECK(seen);
        }
    }
}

// The copies of an LDS histogram: nearly all voxels in one bin are as slow as
// that bin's words are few, so large boxes have the copies that fit.
static void histogram_copies()
{
    struct { int lg, bins, copies; } cases[] = {
        {20, 1024, 4},  {23, 4096, 2},  {23, 8192, 1},  {24, 4096, 4},  {24, 8192, 2},
        {24, 16384, 2}, {25, 16384, 2}, {26, 1024, 8},  {26, 4096, 8},  {26, 5000, 4},
        {26, 8192, 4},  {26, 8446, 4},  {26, 8447, 2},  {26, 16384, 2}, {26, 16894, 2},
        {28, 4096, 8},  {28, 8192, 4},  {28, 16384, 2}, {28, 32768, 1}, {32, 8192, 4}};
    float *x = device_floats((size_t)1 << 32);
    for (auto &c : cases)
        for (int kind : {CUBE_Q_HIST, CUBE_Q_FUSED}) {
            const int64_t dims[5] = {(int64_t)1 << c.lg, 1, 1, 0, 0};
            char plan[512], want[32];
            CHECK(cube_describe_plan(x, dims, kind, c.bins, plan, sizeof plan) == CUBE_OK);
            snprintf(want, sizeof want, "\"copies\": %d,", c.copies);
            if (!strstr(plan, want)) {
                printf("2^%d voxels, %d bins: %s, not %s\n", c.lg, c.bins, plan, want);
                exit(1);
            }
        }
}

// The blocks' rows of counts (32 MiB) are allocated by the first pass that
// writes them, and by no other.
static void rows_memory()
{
    const size_t rows = (size_t)32 << 20;
    const int64_t small[5] = {(1 << 20) - 1, 1, 1, 0, 0}, large[5] = {1 << 20, 1, 1, 0, 0},
                  huge[5] = {(1 << 24) + 1, 1, 1, 0, 0};
    float *x = device_floats((1 << 24) + 1);
    cube_stats_t *out = (cube_stats_t *)take(sizeof *out);
    uint64_t *c = (uint64_t *)take((65536 + 3) * 8);
    auto has = [&] {
        return std::count(g_mallocs.begin(), g_mallocs.end(), rows) != 0;
    };
    auto hist = [&](const int64_t *dims, int bins, bool fused) {
        g_launches.clear();
        CHECK((fused ? cube_stats_hist_async(x, dims, -1.f, 1.f, bins, out, c, STREAM)
                     : cube_hist_async(x, dims, -1.f, 1.f, bins, c, STREAM)) == CUBE_OK);
        CHECK(g_launches[0].is_pass);
        return g_launches[0].pass.dump != nullptr;
    };
    for (bool fused : {false, true}) {
        CHECK(!hist(large, 8191, fused) && !hist(huge, 8192, fused) && !hist(huge, 16383, fused));
        CHECK(!hist(small, 32769, fused) && !hist(small, 65536, fused) && !has());
        CHECK(cube_set_launch(0, 64, 0, 0) == CUBE_OK);       // an explicit grid
        CHECK(!hist(large, 65536, fused) && !has());
        CHECK(cube_set_launch(0, 4096, 0, 0) == CUBE_OK);     // more rows than there is room for
        CHECK(!hist(large, 16384, fused) && !has());
        CHECK(cube_set_launch(0, 0, 0, 0) == CUBE_OK);
        cube_set_hist_mode(CUBE_HIST_HOT);
        CHECK(!hist(large, 8192, fused) && !has());
        cube_set_hist_mode(CUBE_HIST_AUTO);
        g_capturing = true;
        CHECK(!hist(large, 8192, fused) && !hist(large, 65536, fused) && !has());
        g_capturing = false;
        CHECK(hist(large, fused ? 65536 : 8192, fused) && has());
        g_mallocs.clear();
        CHECK(hist(large, 8192, fused) && hist(large, 65536, fused) && hist(huge, 16384, fused));
        g_capturing = true;
        CHECK(hist(large, 8192, fused) && hist(large, 65536, fused) && !has());
        g_capturing = false;
        cube_release_stream(STREAM);
        g_mallocs.clear();
    }
}

int main(int argc, char **argv)
{
    static const std::map<std::string, void (*)()> all = {
        {"shared_stream", shared_stream},
        {"host_results", host_results},
        {"lost_results", lost_results},
        {"shared_projection", shared_projection},
        {"projection_without_partials", projection_without_partials},
        {"captured_partials", captured_partials},
        {"projection_kernels", projection_kernels},
        {"projection_slices", projection_slices},
        {"thin_rows", thin_rows},
        {"histogram_copies", histogram_copies},
        {"rows_memory", rows_memory},
    };
    if (argc != 2 || !all.count(argv[1])) return 2;
    all.at(argv[1])();
    puts("ok");
    return 0;
}
