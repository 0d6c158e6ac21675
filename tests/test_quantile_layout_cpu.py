"""The layout arithmetic that the quantile kernels and the host plan share
(cube_quantile_plan.h), compiled with g++ under AddressSanitizer and UBSan: for
every number of prefixes that a pass can have, the tables and histograms fit
their memory, entries are inside their tables and distinct, and the LDS copies
are the most that fit.  No GPU involved."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1111_6661_amd", "csrc")

DRIVER = r"""
#include "cube_quantile_plan.h"
#include <cstdio>
#include <cstdlib>
#include <set>
using namespace cube;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s (wide %d n %d %d %d)\n", __LINE__, #c, \
    wide, n1, n2, n3); std::exit(1); } } while (0)

// A pass of `slots` prefixes with tables of `tab` bytes.
static void fits(int wide, int n1, int n2, int n3, int slots, int width, size_t tab)
{
    CHECK((slots << width) <= QP_COUNTERS && tab <= QP_TAB_MAX && tab % 4 == 0);
    CHECK(((size_t)slots << width) * 4 + tab <= QP_LDS);
    for (int most = 0; most <= 3; ++most) {
        const int c = qp_copies_log2(slots, width, (int)tab, most, (unsigned)QP_LDS);
        CHECK(c >= 0 && c <= most);
        CHECK(((size_t)slots << width << c) * 4 + tab <= QP_LDS);
        CHECK(c == most || ((size_t)slots << width << (c + 1)) * 4 + tab > QP_LDS);
    }
}

// Every column of rows 1..n of a table lies inside it, at a place of its own
// and off row 0, whatever the key's other bits.
static void entries(int wide, int n1, int n2, int n3, int n, int low, int width)
{
    const unsigned bytes = (unsigned)qp_table_bytes(n, width);
    std::vector<unsigned char> seen(bytes, 0);
    for (unsigned g = 1; g <= (unsigned)n; ++g)
        for (unsigned c = 0; c < 1u << width; ++c) {
            const unsigned e = qp_entry(g, (c << low) | ~(((1u << width) - 1u) << low), low, width);
            CHECK(e == qp_entry(g, c << low, low, width));
            CHECK(e >= 1u << width && e < bytes && !seen[e]);
            seen[e] = 1;
        }
}

int main()
{
    for (int n1 = 1; n1 <= QP_RANKS; ++n1)
        for (int m = n1; m <= QP_RANKS; ++m) {
            const int wide = qp_wide(n1, m), n2 = 0, n3 = 0;
            CHECK(wide == (n1 <= 8 && m <= 96));
            int done = 12;
            for (int l = 1; l <= (wide ? 2 : 3); ++l) done += qp_width(wide, l);
            CHECK(done == 32);
        }
    // Prefixes at each level: at least as many as at the one before, at most
    // the ranks.
    for (int wide = 0; wide < 2; ++wide) {
        const int w1 = qp_width(wide, 1), w2 = qp_width(wide, 2), w3 = qp_width(wide, 3);
        const int most = wide ? 96 : QP_RANKS;
        for (int n1 = 1; n1 <= (wide ? 8 : QP_RANKS); ++n1) {
            fits(wide, n1, 0, 0, n1, w1, 4096);
            entries(wide, n1, 0, 0, n1, 20 - w1, w1);
            for (int n2 = n1; n2 <= most; n2 += n2 < 12 || n2 > most - 4 ? 1 : 7) {
                const size_t t2 = (size_t)qp_table_bytes(n1, w1);
                fits(wide, n1, n2, 0, n2, w2, 4096 + t2);
                if (wide) continue;
                entries(wide, n1, n2, 0, n2, 20 - w1 - w2, w2);
                for (int n3 = n2; n3 <= most; n3 += n3 < 12 || n3 > most - 4 ? 1 : 7)
                    fits(wide, n1, n2, n3, n3, w3, 4096 + t2 + (size_t)qp_table_bytes(n2, w2));
            }
        }
    }
    std::puts("ok");
    return 0;
}
"""


def test_layouts(tmp_path):
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined",
                           "-fno-sanitize-recover=all", "-I", CSRC, "-o", str(exe), str(src)])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout + r.stderr


def test_kernels_take_the_shared_functions():
    """The device's layout and lookups have no arithmetic of their own for what
    is checked above."""
    with open(os.path.join(CSRC, "cube_quantile.hip")) as f:
        text = f.read()
    for name, times in (("qp_wide(", 2), ("qp_width(", 1), ("qp_table_bytes(", 2),
                        ("qp_entry(", 5), ("qp_copies_log2(", 1)):
        assert text.count(name) == times, name
