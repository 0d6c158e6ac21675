// cube_project.hip -- projections of a cube along its channel axis.
//
// The case study renders spectral cubes for inspection (Section 2); the maps a
// viewer shows beside the volume reduce the channel axis of every spatial
// pixel: the maximum-intensity projection, the sum of the channels (the
// moment-0 map up to the channel width) and the number of valid channels.
// One streaming read of the cube makes all three.
//
// Lanes own quads of pixels numbered over the image row by row (rows that
// follow each other in memory count as one), Q quads per lane 64 apart, so
// that per channel a wavefront reads Q KB of the image, contiguous along a
// row; long runs keep HBM pages open (a probe of 16 GiB: 5.97 TB/s with 1 KB
// per wavefront and channel, 7.26 with 16 KB).  A quad is one float4 load at
// any alignment; a row's last quad overlaps the one before it, and only its
// own pixels are written.  Q * ZU loads are in flight per lane (ZU channels).
// Each lane walks the channels of its pixels.  The sums are taken in FP64: on
// CDNA4 an FP64 add issues at the rate of an FP32 add, so this costs no more
// than compensated FP32 and is exact to about n * 2^-53.  When the image has
// too few pixels to fill the device the channels are split into slices, each
// slice writes per-pixel partials, and a second kernel merges them in slice
// order, so the result never depends on timing.  Small images, and those that
// quads do not fit (rows under four pixels, or apart by more than 32-bit
// offsets reach), take one pixel per lane (k_project).
#include <string.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <utility>

#include "cube_device.h"

namespace cube {

namespace {

struct ProjArgs {
    const float *ptr;
    int64_t nx, ny, nz, sy, sz;  // rows that follow each other merged into one
    int64_t units;           // lanes' work items: quads, or pixels (k_project)
    int64_t quads_row;       // quads per row
    int64_t per;             // quads per wavefront
    int64_t zps;             // channels per slice
    int32_t slices;
    float *mip;              // outputs, dense nx * ny (any may be null)
    double *mom0;
    uint32_t *nvalid;
    float *p_max;            // slice partials [slices][npix] (slices > 1)
    double *p_sum;
    uint32_t *p_cnt;
};

constexpr int PROJ_THREADS = 256;
constexpr int PROJ_ZU = 4;

struct Pixel {
    float m;
    double s;
    uint32_t n;
    __device__ __forceinline__ void take(float x)
    {
        const bool ok = x == x;
        m = fmaxf(m, __builtin_canonicalizef(x));  // a (quieted) NaN is skipped
        s += (double)(ok ? x : 0.f);
        n += (uint32_t)ok;
    }
};
constexpr Pixel PIXEL_NONE = {-INFINITY, 0.0, 0u};

// Pixel p (of npix) of slice `slice`: the maps, or its partial.
__device__ __forceinline__ void put_pixel(const ProjArgs &a, int64_t p, int slice, const Pixel &v)
{
    if (a.slices == 1) {
        if (a.mip) a.mip[p] = v.n ? v.m : qnan();
        if (a.mom0) a.mom0[p] = v.n ? v.s : (double)qnan();
        if (a.nvalid) a.nvalid[p] = v.n;
    } else {
        const int64_t o = (int64_t)slice * a.nx * a.ny + p;
        a.p_max[o] = v.m;
        a.p_sum[o] = v.s;
        a.p_cnt[o] = v.n;
    }
}

__global__ void __launch_bounds__(PROJ_THREADS) k_project(ProjArgs a)
{
    const int64_t p = (int64_t)blockIdx.x * PROJ_THREADS + threadIdx.x;
    if (p >= a.units) return;
    const int64_t y = p / a.nx;
    const int64_t x = p - y * a.nx;
    const int64_t z0 = (int64_t)blockIdx.y * a.zps;
    const int64_t z1 = min(a.nz, z0 + a.zps);
    const float *q = a.ptr + y * a.sy + x + z0 * a.sz;
    Pixel v = PIXEL_NONE;
    int64_t z = z0;
    for (; z + PROJ_ZU <= z1; z += PROJ_ZU) {
        float t[PROJ_ZU];
#pragma unroll
        for (int j = 0; j < PROJ_ZU; ++j) t[j] = __builtin_nontemporal_load(q + j * a.sz);
#pragma unroll
        for (int j = 0; j < PROJ_ZU; ++j) v.take(t[j]);
        q += PROJ_ZU * a.sz;
    }
    for (; z < z1; ++z) {
        v.take(__builtin_nontemporal_load(q));
        q += a.sz;
    }
    put_pixel(a, p, (int)blockIdx.y, v);
}

// Wavefront w owns a.per quads from a.per * w on (the last one the image's last
// a.per: what it shares with its neighbour both write alike), lane l the quads
// 64 k + l of them.  All wavefronts have the same work and the same number
// falls to every CU: with 64 Q quads each, 1057 wavefronts took 537 us where
// 1024 took 362 (a CU with two blocks sets the end).  Bound by HBM from about
// 2^26 voxels on.  Measured (async calls) on a 1187 x 911 x 512 cut-out of
// 2048-wide rows: 490 us with one pixel per lane, 345 with quads; on 300 dense
// planes of 2035 x 1599: 848 -> 570.
// ONE_ROW: the image is one row, every quad but the last at its plain place.
template <int Q, int ZU, bool ONE_ROW>
__global__ void __launch_bounds__(PROJ_THREADS) k_project_quads(ProjArgs a)
{
    // Four neighbouring wavefronts per block: they stay on one CU and read
    // side by side (blocks of one: 2418 us on 2048 x 2048 x 1024, four: 2380).
    const int lane = threadIdx.x & 63;
    const int64_t wave = (int64_t)blockIdx.x * (PROJ_THREADS / 64) +
                         __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (wave * a.per >= a.units) return;
    const int64_t qb = min(wave * a.per, a.units - a.per);
    // The wavefront's first row, and each quad's place from its start.
    const int64_t y0 = ONE_ROW ? 0 : qb / a.quads_row;
    const uint32_t c0 = ONE_ROW ? 0u : (uint32_t)(qb - y0 * a.quads_row);
    const uint32_t row = (uint32_t)min(a.quads_row, (int64_t)0xffffffff);
    auto place = [&](int k, uint32_t *dy, uint32_t *x, uint32_t *own) {
        const uint32_t i = (uint32_t)(64 * k + lane), last = (uint32_t)a.per - 1u;
        const uint32_t c = c0 + min(i, last);
        if (ONE_ROW) {  // x from quad qb on; the image's last quad ends with it
            *dy = 0u;
            *x = (uint32_t)min((int64_t)4 * c, a.nx - 4 - 4 * qb);
            *own = 4u * c - *x;
        } else {
            *dy = c / row;
            const uint32_t col = c - *dy * row;
            *x = min(4u * col, (uint32_t)a.nx - 4u);
            *own = 4u * col - *x;  // the quad's first own pixel
        }
        if (i > last) *own = 4u;
    };
    uint32_t off[Q];
    Pixel v[Q][4];
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        uint32_t dy, x, own;
        if (ONE_ROW && k < Q - 1) {
            off[k] = (uint32_t)(lane * 16 + k * 1024);
        } else {
            place(k, &dy, &x, &own);
            off[k] = (dy * (uint32_t)a.sy + x) * 4u;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) v[k][j] = PIXEL_NONE;
    }
    const int64_t z0 = (int64_t)blockIdx.y * a.zps;
    const int64_t z1 = min(a.nz, z0 + a.zps);
    const char *base =
        (const char *)(a.ptr + (ONE_ROW ? 4 * qb : y0 * a.sy) + z0 * a.sz);
    const int64_t step = a.sz * 4;
    auto load = [&](f4 (&t)[Q], const char *b) {
#pragma unroll
        for (int k = 0; k < Q; ++k) t[k] = __builtin_nontemporal_load((const f4u *)(b + off[k]));
    };
    auto take = [&](const f4 (&t)[Q]) {
#pragma unroll
        for (int k = 0; k < Q; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) v[k][j].take(t[k][j]);
    };
    int64_t z = z0;
    if (ZU > 1)
        for (; z + ZU <= z1; z += ZU) {
            f4 t[ZU][Q];
#pragma unroll
            for (int u = 0; u < ZU; ++u) load(t[u], base + u * step);
            // All loads first: the scheduler otherwise takes some of them one
            // by one to save registers (twice the time with four quads).
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < ZU; ++u) take(t[u]);
            base += ZU * step;
        }
    for (; z < z1; ++z) {
        f4 t[Q];
        load(t, base);
        take(t);
        base += step;
    }
#pragma unroll
    for (int k = 0; k < Q; ++k) {
        uint32_t dy, x, own;
        place(k, &dy, &x, &own);
        const int64_t p = (ONE_ROW ? 4 * qb : (y0 + dy) * a.nx) + x;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if ((uint32_t)j >= own) put_pixel(a, p + j, (int)blockIdx.y, v[k][j]);
    }
}

template <int Q>
void launch_quads(const ProjArgs &a, hipStream_t s)
{
    // Channels in flight: about 16 loads with few wavefronts per CU; four
    // with one quad per lane and many (600 x 600 x 256: 72 us, eight: 80).
    constexpr int ZU = Q >= 9 ? 1 : (Q >= 5 ? 2 : (Q == 2 ? 8 : 4));
    const int64_t waves = (a.units + a.per - 1) / a.per;
    const dim3 grid((unsigned)((waves * 64 + PROJ_THREADS - 1) / PROJ_THREADS),
                    (unsigned)a.slices);
    if (a.ny == 1)
        hipLaunchKernelGGL((k_project_quads<Q, ZU, true>), grid, dim3(PROJ_THREADS), 0, s, a);
    else
        hipLaunchKernelGGL((k_project_quads<Q, ZU, false>), grid, dim3(PROJ_THREADS), 0, s, a);
}

// The choice of kernel and slices, measured with cold caches against every
// other (1579 shapes of 24 to 2040 pixels a side and 16 to 1000 channels, in
// cut-outs and whole): 1.9 % over the best of each, on the average.

// Few pixels and channels take one pixel per lane: a lane's own work, a quarter
// of a quad's, is then the bound.  256 x 256 x 32: 10.2 us against 12.2 by
// quads, 450 x 450 x 32 11.9 and 13.7; 300 x 300 x 256 26.6 and 26.2, 400 x 400
// x 128 24.4 and 25.3.  So do up to 256 channels of images that give some CUs
// two blocks of quads and most one (550 x 550 x 256: 64.2 against 67.2); six to
// nine wavefronts of one quad per lane on a CU do well by themselves (a 680 x 680
// cut-out of 24 channels: 15.8 against 14.5 by quads, of 16: 11.9 and 12.6).
bool small_projection(int64_t quad_waves, int64_t nz, int64_t cus)
{
    if (quad_waves > 6 * cus && quad_waves <= 9 * cus) return nz <= 16;
    return quad_waves * nz <= 288 * cus ||
           (quad_waves > 4 * cus && quad_waves <= 5 * cus && nz <= 256);
}

// Slices of the channels, for images of few wavefronts.  One quad per lane: as
// many as keep two blocks of four wavefronts per CU at most (640 x 640 x 256,
// 1600 wavefronts: one slice 77 us, two 93; 300 x 300 x 1000, 352: five 69,
// six 82), each of 48 channels or more (the merge is a launch of 4 us).
int64_t quad_slices(int64_t waves, int64_t nz, int64_t cus)
{
    const int64_t n = std::min(std::min(nz / 48, 8 * cus / waves), (int64_t)64);
    // From four blocks for three CUs on the second slice pays for long columns
    // (580 x 580 x 1000: 234 us against 253).
    if (n <= 1 && 2 * waves <= 11 * cus && nz >= 400) return 2;
    return std::max(n, (int64_t)1);
}

// One pixel per lane: 18 wavefronts per CU, 20 channels or more, and not more
// slices than the merge is worth (100 x 100 x 512: 16, 19 us; 32, 22 us).
int64_t pixel_slices(int64_t waves, int64_t nz, int64_t cus)
{
    const int64_t most = std::min(std::max(nz / 64, (int64_t)16), (int64_t)64);
    return std::max(std::min(std::min(nz / 20, 18 * cus / waves), most), (int64_t)1);
}

// Merge the slice partials of every pixel in slice order.
__global__ void __launch_bounds__(PROJ_THREADS) k_project_merge(ProjArgs a)
{
    const int64_t npix = a.nx * a.ny;
    const int64_t p = (int64_t)blockIdx.x * PROJ_THREADS + threadIdx.x;
    if (p >= npix) return;
    float m = -INFINITY;
    double s = 0.0;
    uint32_t n = 0u;
    for (int k = 0; k < a.slices; ++k) {
        const int64_t o = (int64_t)k * npix + p;
        m = fmaxf(m, a.p_max[o]);
        s += a.p_sum[o];
        n += a.p_cnt[o];
    }
    if (a.mip) a.mip[p] = n ? m : qnan();
    if (a.mom0) a.mom0[p] = n ? s : (double)qnan();
    if (a.nvalid) a.nvalid[p] = n;
}

__global__ void k_project_empty(ProjArgs a)
{
    const int64_t npix = a.nx * a.ny;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < npix;
         p += (int64_t)gridDim.x * blockDim.x) {
        if (a.mip) a.mip[p] = qnan();
        if (a.mom0) a.mom0[p] = (double)qnan();
        if (a.nvalid) a.nvalid[p] = 0u;
    }
}

// Slice partials, one buffer per (device, stream), grown on demand.
struct ProjScratch {
    void *ptr = nullptr;
    size_t bytes = 0;
    bool captured = false;      // a graph holds its address
    std::vector<void *> kept;   // outgrown buffers that graphs hold (each under half the next)
    // Held from the buffer's choice until the merge is queued: another thread's
    // projection on the stream would overwrite the partials, or free them.
    std::mutex queue;
};
std::mutex g_pmu;
std::map<std::pair<int, hipStream_t>, ProjScratch> g_pscratch;

ProjScratch &scratch_of(hipStream_t s)
{
    int dev = 0;
    hipGetDevice(&dev);
    std::lock_guard<std::mutex> lk(g_pmu);
    return g_pscratch[std::make_pair(dev, s)];
}

// Whether `ps` (of stream s, its lock held) has room for `bytes`, made if need
// be.  Not while the stream captures: nothing can be allocated or waited for.
bool have_scratch(ProjScratch &ps, hipStream_t s, size_t bytes)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    bool capturing = false;
    if (s && (hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone)) {
        (void)hipGetLastError();
        capturing = true;
    }
    if (ps.bytes >= bytes) {
        ps.captured |= capturing;
        return true;
    }
    if (capturing) return false;
    if (ps.captured) bytes = std::max(bytes, 2 * ps.bytes);
    void *p = nullptr;
    // Earlier work on this stream may still read the old buffer.
    if (hipMalloc(&p, bytes) != hipSuccess ||
        (ps.ptr && !ps.captured && hipStreamSynchronize(s) != hipSuccess)) {
        (void)hipGetLastError();
        hipFree(p);
        return false;
    }
    if (ps.captured)
        ps.kept.push_back(ps.ptr);
    else
        hipFree(ps.ptr);
    ps.ptr = p;
    ps.bytes = bytes;
    ps.captured = false;
    return true;
}

// An output map must be device memory holding `bytes`, aligned to `align`.
int check_output(const void *p, size_t bytes, uintptr_t align, const char *what)
{
    if (!p) return CUBE_OK;
    if ((uintptr_t)p % align)
        return fail(CUBE_EINVAL, "%s is not %d-byte aligned", what, (int)align);
    Box b;
    b.ptr = (const float *)p;
    b.nx = (int64_t)(bytes / 4);
    b.ny = b.nz = 1;
    b.sy = b.nx;
    b.sz = b.nx;
    b.n = (uint64_t)b.nx;
    const int rc = check_box_device(&b);
    if (rc) return fail(rc, "%s: %s", what, cube_last_error());
    return CUBE_OK;
}

}  // namespace

void project_release()
{
    std::lock_guard<std::mutex> lk(g_pmu);
    int cur = 0;
    hipGetDevice(&cur);
    for (auto &kv : g_pscratch) {
        // The stream may be gone: wait for the whole device instead.
        hipSetDevice(kv.first.first);
        hipDeviceSynchronize();
        hipFree(kv.second.ptr);
        for (void *p : kv.second.kept) hipFree(p);
    }
    hipSetDevice(cur);
    g_pscratch.clear();
}

}  // namespace cube

using namespace cube;

extern "C" {

int cube_project(const float *ptr, const int64_t *dims, float *mip, double *mom0,
                 uint32_t *nvalid, void *stream)
{
    CUBE_GUARD_BEGIN
    if (!mip && !mom0 && !nvalid) return fail(CUBE_EINVAL, "every output is NULL");
    Box b;
    int rc = check_box(ptr, dims, &b);
    if (rc) return rc;
    if (b.nz >= ((int64_t)1 << 32)) return fail(CUBE_EINVAL, "more than 2^32 - 1 channels");
    const int64_t npix = b.nx * b.ny;
    if (npix == 0) return CUBE_OK;
    if ((rc = check_output(mip, (size_t)npix * 4, 4, "mip")) ||
        (rc = check_output(mom0, (size_t)npix * 8, 8, "mom0")) ||
        (rc = check_output(nvalid, (size_t)npix * 4, 4, "nvalid")))
        return rc;
    if ((rc = check_box_device(&b))) return rc;
    hipStream_t s = (hipStream_t)stream;
    ProjArgs a;
    memset(&a, 0, sizeof a);
    a.ptr = b.ptr;
    a.nx = b.nx;
    a.ny = b.ny;
    a.nz = b.nz;
    a.sy = b.ny > 1 ? b.sy : b.nx;
    a.sz = b.nz > 1 ? b.sz : 0;
    a.mip = mip;
    a.mom0 = mom0;
    a.nvalid = nvalid;
    hipError_t e;
    if (b.nz == 0) {
        hipLaunchKernelGGL(k_project_empty, dim3(1024), dim3(256), 0, s, a);
        e = hipGetLastError();
        return e == hipSuccess ? CUBE_OK : hip_fail(e, "projection launch");
    }
    // Rows that follow each other are one row.
    if (a.ny > 1 && a.sy == a.nx) {
        a.nx = a.sy = npix;
        a.ny = 1;
    }
    a.quads_row = (a.nx + 3) / 4;
    const int64_t quads = a.quads_row * a.ny;
    // Quads while a wavefront's offsets from its first row fit 32 bits; in one
    // row they are from its own first quad, 16 KB at most.
    const bool fits =
        a.nx >= 4 && (a.ny == 1 || (a.nx < ((int64_t)1 << 31) &&
                                    64 * 16 / a.quads_row + 2 < ((int64_t)1 << 30) / a.sy));
    const int64_t cus = cu_count(), nz = b.nz;
    const int64_t quad_waves = (quads + 63) / 64;  // with one quad per lane
    const bool quad = fits && !small_projection(quad_waves, nz, cus);
    a.units = quad ? quads : npix;
    int64_t slices = 1;
    if (quad && quad_waves > 9 * cus) {
        // Equal shares for every CU: a multiple of one block of four wavefronts
        // per CU, as few as up to 16 quads per lane allow (each holds 16 Q
        // registers of state).
        const int64_t most = 4 * cus * 64 * 16;
        const int64_t waves = 4 * cus * ((a.units + most - 1) / most);
        a.per = (a.units + waves - 1) / waves;
    } else {
        a.per = std::min<int64_t>(64, a.units);
        slices = quad ? quad_slices(quad_waves, nz, cus)
                      : pixel_slices((a.units + 63) / 64, nz, cus);
    }
    const int Q = (int)((a.per + 63) / 64);
    a.zps = (nz + slices - 1) / slices;
    a.slices = (int32_t)((nz + a.zps - 1) / a.zps);
    // Without memory for their partials there is one slice.
    std::unique_lock<std::mutex> queue;
    if (a.slices > 1) {
        ProjScratch &ps = scratch_of(s);
        queue = std::unique_lock<std::mutex>(ps.queue);
        const size_t per = (size_t)npix * (size_t)a.slices;
        if (have_scratch(ps, s, per * 16)) {
            a.p_sum = (double *)ps.ptr;
            a.p_max = (float *)((char *)ps.ptr + per * 8);
            a.p_cnt = (uint32_t *)((char *)ps.ptr + per * 12);
        } else {
            a.zps = b.nz;
            a.slices = 1;
        }
    }
    if (!quad) {
        hipLaunchKernelGGL(k_project,
                           dim3((unsigned)((a.units + PROJ_THREADS - 1) / PROJ_THREADS),
                                (unsigned)a.slices),
                           dim3(PROJ_THREADS), 0, s, a);
    } else {
        using Launch = void (*)(const ProjArgs &, hipStream_t);
        static const Launch by_q[16] = {
            launch_quads<1>,  launch_quads<2>,  launch_quads<3>,  launch_quads<4>,
            launch_quads<5>,  launch_quads<6>,  launch_quads<7>,  launch_quads<8>,
            launch_quads<9>,  launch_quads<10>, launch_quads<11>, launch_quads<12>,
            launch_quads<13>, launch_quads<14>, launch_quads<15>, launch_quads<16>};
        by_q[Q - 1](a, s);  // Q <= 16
    }
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "projection launch");
    if (a.slices > 1) {
        hipLaunchKernelGGL(k_project_merge, dim3((unsigned)((npix + PROJ_THREADS - 1) / PROJ_THREADS)),
                           dim3(PROJ_THREADS), 0, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "projection merge");
    }
    return CUBE_OK;
    CUBE_GUARD_END
}

}  // extern "C"
