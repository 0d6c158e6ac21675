"""The packing of short rows (cube_rows.h), walked lane by lane on the CPU.

For every plan, the lanes of the blocks that share the rows must visit each
voxel exactly once and load nothing outside a row, whatever the row length,
pitch, alignment, split of the rows and block shape.
"""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1111_6661_amd", "csrc")

DRIVER = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "cube_rows.h"
using namespace cube;
#define CHECK(c) do { if (!(c)) { printf("line %d: %s (len %ld ny %ld nz %ld sy %ld sz %ld mis %d "\
    "threads %d unroll %d cut %u)\n", __LINE__, #c, (long)len, (long)ny, (long)nz, (long)sy, \
    (long)sz, mis, threads, unroll, cut); exit(1); } } while (0)

static long plans = 0;

static void walk(int64_t len, int64_t ny, int64_t nz, int64_t sy, int64_t sz, int mis, int threads,
                 int unroll, uint32_t cut)
{
    const RowPack k = row_pack(len, ny, nz, sy, sz, 1, mis, threads, unroll);
    if (!k.cb) return;
    ++plans;
    const uint32_t rows = (uint32_t)(ny * nz);
    const int64_t end = (nz - 1) * sz + (ny - 1) * sy + len;
    std::vector<float> mem((size_t)end);            // the box's own extent
    std::vector<unsigned char> seen((size_t)end, 0);
    const float *base = mem.data();
    CHECK(k.rb >= 1 && k.rb * k.cb <= threads && k.cg <= unroll && unroll % k.cg == 0);
    for (uint32_t r0 = 0; r0 < rows; r0 += cut) {
        const uint32_t r1 = r0 + cut < rows ? r0 + cut : rows;
        const uint32_t tiles = row_tiles(k, r0, r1, unroll);
        for (int t = 0; t < threads; ++t) {
            const uint32_t lr = (uint32_t)t / k.cb, lc = (uint32_t)t - lr * k.cb;
            RowLane l = row_lane(k, base, sy, sz, (uint32_t)ny, r0, r1, lr);
            for (uint32_t i = 0; i < tiles; ++i)
                for (int v = 0; v < unroll; ++v) {
                    const int j = v & (k.cg - 1);
                    if (l.row < l.row_end) {
                        int s, d;
                        row_vector(k, (int)len, lc, j, &s, &d);
                        CHECK(s >= 0 && s + 4 <= len);
                        const int64_t row = (int64_t)(l.row / ny) * sz + (l.row % ny) * sy;
                        CHECK(l.p - base == row);
                        if (k.h < 4 && d == 0 && s)    // an aligned load
                            CHECK((row + s - mis) % 4 == 0);
                        for (int e = 0; e < 4; ++e)
                            if (row_own(e, d)) ++seen[(size_t)(row + s + e)];
                    }
                    if (((v + 1) & (k.cg - 1)) == 0) row_advance(k, (uint32_t)ny, l);
                }
            CHECK(l.row >= r1);                     // nothing left
        }
    }
    long visited = 0;
    for (int64_t z = 0; z < nz; ++z)
        for (int64_t y = 0; y < ny; ++y)
            for (int64_t x = 0; x < len; ++x) {
                CHECK(seen[(size_t)(z * sz + y * sy + x)] == 1);
                ++visited;
            }
    long all = 0;
    for (unsigned char c : seen) all += c;
    CHECK(all == visited);
}

int main()
{
    const int lens[] = {4, 5, 6, 7, 8, 9, 15, 16, 17, 61, 63, 64, 65, 255, 257, 1023, 1024, 1025,
                        1187, 2047, 2049, 4095, 4096, 4097, 8191, 8193, 16383, 16384, 16385};
    for (int threads : {256, 512, 1024})
        for (int unroll : {2, 4})
            for (int len : lens)
                for (int ny : {1, 2, 3, 47, 300})
                    for (int nz : {1, 2, 5}) {
                        if ((long)len * ny * nz > 60000) continue;
                        for (int gap : {0, 1, 2, 3, 4, 8})
                            for (int mis : {0, 1, 2, 3}) {
                                const int64_t sy = len + gap, sz = sy * ny + (gap & 1 ? 3 : gap);
                                const uint32_t cuts[] = {1, 3, 64, 1u << 20};
                                walk(len, ny, nz, ny == 1 ? 0 : sy, nz == 1 ? 0 : sz, mis,
                                     threads, unroll, cuts[(len + gap + mis + ny) % 4]);
                            }
                    }
    // not packed: cut rows, a single row, rows under one vector, a whole tile
    if (row_pack(100, 10, 10, 128, 2000, 2, 0, 256, 4).cb) return 2;
    if (row_pack(100, 1, 1, 0, 0, 1, 0, 256, 4).cb) return 3;
    if (row_pack(3, 10, 10, 128, 2000, 1, 0, 256, 4).cb) return 4;
    if (row_pack(4097, 10, 10, 8000, 90000, 1, 0, 256, 4).cb) return 5;
    if (!row_pack(4096, 10, 10, 8000, 90000, 1, 0, 256, 4).cb) return 6;
    printf("plans %ld\n", plans);
    return plans > 1000 ? 0 : 7;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("rows")
    src, exe = d / "walk.cpp", d / "walk"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC, "-o", str(exe), str(src)])
    return str(exe)


def test_rows_visited_once_and_in_bounds(driver):
    r = subprocess.run([driver], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
