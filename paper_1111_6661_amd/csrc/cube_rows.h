// cube_rows.h -- how the lanes of a block share short rows: the plan (host),
// and each lane's rows and vectors (device).  Plain C++ with no GPU call, so
// that a CPU test can walk every lane of a plan.
//
// A row of a cut-out is often far shorter than the tile a block reads at a
// time, and a block that takes one row at a time keeps most of its lanes idle
// and one load in flight per lane.  Packed, the lanes of a block form rb rows
// of cb columns; a lane owns the same columns (float4 vectors lc, lc + cb, ...
// of cg column groups) of every rb-th row.
//
// A row's first vector takes the h voxels up to the first 16-byte boundary
// when every row has the same alignment; else h = 4 and loads are at 4-byte
// alignments (measured on 4 GiB: 6.6 TB/s against 7.1 for aligned float4
// loads).  The other vectors take four voxels each.  The first and the last
// are loaded inside the row, overlapping their neighbours, and the overlap is
// masked off, so no load leaves the row.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define CUBE_HD __host__ __device__ __forceinline__
#else
#define CUBE_HD inline
#endif

namespace cube {

struct RowPack {
    int32_t cb, rb, cg;  // columns, rows, column groups (1, 2 or 4); cb == 0: not packed
    int32_t h;           // voxels of a row's first vector (1..4)
    int32_t dy, pad;     // rows advanced within a plane per step of rb rows
    int64_t inc, wrap;   // pointer steps: rb rows on, and past a plane's end
};

// The plan for blocks of `threads` threads that take `unroll` vectors per lane
// per tile; `mis`: voxels from the first row's start to a 16-byte boundary
// (0..3).  cb == 0 where rows are cut (segs > 1), single, under one vector, or
// as long as a block tile (the unpacked scan then reads mostly whole tiles).
inline RowPack row_pack(int64_t row_len, int64_t ny, int64_t nz, int64_t sy, int64_t sz,
                        int64_t segs, int mis, int threads, int unroll)
{
    RowPack p = {0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t rows = ny * nz;
    if (segs != 1 || rows < 2 || rows > 0x7fffffff || row_len < 4) return p;
    if (row_len > (int64_t)4 * threads * unroll) return p;
    const bool same = (ny == 1 || sy % 4 == 0) && (nz == 1 || sz % 4 == 0);
    const int h = same && mis ? mis : 4;
    const int vecs = 1 + (int)((row_len - h + 3) / 4);  // vectors per row
    // The column groups that keep the most lanes busy; fewer groups (longer
    // contiguous reads per wavefront) unless more gain over 3 %.
    double best = 0.0;
    for (int cg = 1; cg <= unroll; cg *= 2) {
        const int cb = (vecs + cg - 1) / cg;
        if (cb > threads) continue;
        const int rb = threads / cb;
        const double use = (double)rb * vecs / ((double)threads * cg);
        if (use > best * 1.03) {
            best = use;
            p.cb = cb;
            p.rb = rb;
            p.cg = cg;
        }
    }
    if (!p.cb) return p;
    p.h = h;
    p.dy = (int32_t)(p.rb % ny);
    p.inc = (p.rb / ny) * sz + p.dy * sy;
    p.wrap = sz - ny * sy;
    return p;
}

// One lane's place: its next row (valid while row < row_end) and that row's
// first voxel.
struct RowLane {
    const float *p;
    uint32_t y, row, row_end;
};

CUBE_HD RowLane row_lane(const RowPack &k, const float *ptr, int64_t sy, int64_t sz, uint32_t ny,
                         uint32_t r0, uint32_t r1, uint32_t lr)
{
    const uint32_t z0 = r0 / ny;                           // uniform over the block
    const uint32_t yl = r0 - z0 * ny + lr, zl = yl / ny;
    RowLane l;
    l.y = yl - zl * ny;
    l.row = r0 + lr;
    l.row_end = lr < (uint32_t)k.rb ? r1 : 0u;             // lanes past the last whole row idle
    l.p = ptr + (int64_t)(z0 + zl) * sz + (int64_t)l.y * sy;
    return l;
}

CUBE_HD void row_advance(const RowPack &k, uint32_t ny, RowLane &l)
{
    l.row += (uint32_t)k.rb;
    l.y += (uint32_t)k.dy;
    l.p += k.inc;
    if (l.y >= ny) {
        l.y -= ny;
        l.p += k.wrap;
    }
}

// Where column lc's vector of column group j is loaded in its row: s, and
// d = s minus the voxel the vector should start at.  Voxel i of the load is
// the lane's own when row_own(i, d).
CUBE_HD void row_vector(const RowPack &k, int len, uint32_t lc, int j, int *s, int *d)
{
    const int c = k.h - 4 + 4 * (int)(lc + (uint32_t)(j * k.cb));
    const int lo = c < 0 ? 0 : c;
    *s = lo < len - 4 ? lo : len - 4;
    *d = *s - c;
}
CUBE_HD bool row_own(int i, int d) { return (uint32_t)(i + d) < 4u; }

// Tiles of `unroll` vectors per lane that cover rows [r0, r1).
CUBE_HD uint32_t row_tiles(const RowPack &k, uint32_t r0, uint32_t r1, int unroll)
{
    const uint32_t steps = (r1 - r0 + (uint32_t)k.rb - 1) / (uint32_t)k.rb;
    const uint32_t per = (uint32_t)(unroll / k.cg);
    return (steps + per - 1) / per;
}

}  // namespace cube
