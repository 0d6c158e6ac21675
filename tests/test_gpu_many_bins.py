"""Histograms on both sides of the lines between the forms of many bins (GPU):
from 8192 bins on a second kernel finishes the bins; up to 2^24 voxels, and
from 16384 bins on, the blocks write rows of counts that it adds up; more than
32768 bins of 2^20 voxels and more are counted in 16 bits in LDS.  Counts must
equal the oracle's exactly."""
import numpy as np
import pytest

import oracle
from tests.parity import assert_stats_match

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LO, HI = -2.0, 2.0


@pytest.fixture(scope="module")
def cs():
    import paper_1111_6661_amd as cs
    assert torch.cuda.is_available()
    cs.load()
    return cs


@pytest.fixture(scope="module")
def boxes():
    """{(kind, n): (host, device, statistics)}; most voxels in one bin, or noise."""
    out = {}
    for n in ((1 << 20) - 1, 1 << 20, 1 << 24, (1 << 24) + 1):
        for kind in ("noise", "one"):
            a = np.random.default_rng(n).standard_normal(n, dtype=np.float32)
            if kind == "one":
                a[a > -1.5] = 0.7
            a[::1001] = np.nan
            out[kind, n] = (a, torch.from_numpy(a).cuda(), oracle.stats(a))
    return out


@pytest.mark.parametrize("nbins", [8191, 8192, 16383, 16384, 32768, 32769])
@pytest.mark.parametrize("n", [(1 << 20) - 1, 1 << 20, 1 << 24, (1 << 24) + 1])
@pytest.mark.parametrize("kind", ["noise", "one"])
def test_forms_of_many_bins(cs, boxes, kind, n, nbins):
    a, t, ref = boxes[kind, n]
    want = oracle.hist(a, LO, HI, nbins)
    for _ in range(2):                  # the accumulators were left at zero
        assert np.array_equal(cs.hist(t, LO, HI, nbins), want)
    st, got = cs.stats_hist(t, LO, HI, nbins)
    assert np.array_equal(got, want)
    assert_stats_match(st, ref, f"{kind} {n} {nbins}")
    st, got = cs.stats_hist_minmax(t, nbins)
    assert np.array_equal(got, oracle.hist(a, ref.min, ref.max, nbins))


@pytest.mark.parametrize("nbins", [8192, 16383, 16384])
def test_captured_without_rows(cs, boxes, nbins):
    """A stream without room for the rows is captured: 32-bit counters, flushed
    by atomics, finished by the second kernel; every replay."""
    a, t, ref = boxes["noise", 1 << 20]
    want = oracle.hist(a, LO, HI, nbins)
    ptr, d = cs.box_of(t)
    c = torch.zeros(nbins + 3, dtype=torch.int64, device="cuda")
    out = torch.zeros(64, dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    cs.cube_hist_async(ptr, d, LO, HI, 64, c.data_ptr(), s.cuda_stream)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        cs.cube_stats_hist_async(ptr, d, LO, HI, nbins, out.data_ptr(), c.data_ptr(),
                                 s.cuda_stream)
    for k in range(3):
        c.fill_(-1)
        cs.hist(t, LO, HI, nbins)       # eager, with rows, on another stream
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(c.cpu().numpy().astype(np.uint64), want), k
        assert_stats_match(cs.Stats.from_bytes(out.cpu().numpy().tobytes()), ref, f"replay {k}")
    del g
    cs.cube_release_stream(s.cuda_stream)
