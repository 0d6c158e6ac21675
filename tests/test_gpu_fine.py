"""Histograms of many bins on the GPU: 16-bit LDS counters (more than 32768
bins) and the blocks' rows summed by a second kernel (2048 bins and more).
Counts must equal the oracle's exactly."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    import paper_1111_6661_amd as cs
    assert torch.cuda.is_available()
    cs.load()
    return cs


def data(kind, n):
    rng = np.random.default_rng(n + len(kind))
    a = rng.standard_normal(n).astype(np.float32)
    if kind == "constant":        # one counter: 0x8000 reached all the time
        a[:] = 0.25
    elif kind == "two":           # both halves of one word (bins 100 and 100 + 32768 of 65536)
        a[:] = np.where(rng.random(n) < 0.5, -2 + 4 * 100.5 / 65536, -2 + 4 * 32868.5 / 65536)
    elif kind == "edges":
        a[::3] = 2.0
        a[1::3] = -2.0
    a[rng.random(n) < 0.01] = np.nan
    return a


@pytest.mark.parametrize("nbins", [2047, 2048, 32768, 32769, 40000, 65535, 65536])
@pytest.mark.parametrize("kind", ["normal", "constant", "two", "edges"])
def test_many_bins(cs, nbins, kind):
    for n in ((1 << 20) - 1, (1 << 20), (1 << 22) + 13):
        a = data(kind, n)
        t = torch.from_numpy(a).cuda()
        want = oracle.hist(a, -2.0, 2.0, nbins)
        assert np.array_equal(cs.hist(t, -2.0, 2.0, nbins), want), (n, kind)
        st, got = cs.stats_hist(t, -2.0, 2.0, nbins)
        assert np.array_equal(got, want), (n, kind)
        prev = cs.cube_set_partition(16)
        try:
            assert np.array_equal(cs.hist(t, -2.0, 2.0, nbins), want), (n, kind)
            assert np.array_equal(cs.stats_hist(t, -2.0, 2.0, nbins)[1], want), (n, kind)
        finally:
            cs.cube_set_partition(prev)


def test_minmax_of_many_bins(cs):
    a = data("normal", 3_000_001)
    t = torch.from_numpy(a).cuda()
    st, got = cs.stats_hist_minmax(t, 65536)
    assert np.array_equal(got, oracle.hist(a, st.min, st.max, 65536))
    t.fill_(float("nan"))                      # no valid voxel: bins zero
    st, got = cs.stats_hist_minmax(t, 65536)
    assert got[:-1].sum() == 0 and got[-1] == a.size
    t[5] = float("inf")                        # an invalid range: bins zero, an error
    with pytest.raises(cs.CubeError):
        cs.stats_hist_minmax(t, 65536)
    t.fill_(1.0)
    assert cs.hist(t, 0.0, 2.0, 65536).sum() == a.size   # the accumulators were left at zero


def test_host_chunks_add_up(cs):
    a = data("normal", 3 * (1 << 20)).reshape(3, 1024, 1024)
    _, got = cs.host_query(a, cs.CUBE_Q_HIST, 65536, -2.0, 2.0, chunk_voxels=1 << 20)
    assert np.array_equal(got, oracle.hist(a, -2.0, 2.0, 65536))


def test_capture_without_a_buffer(cs):
    """A stream known to the library but without the buffer for the blocks'
    rows is captured: the pass must not allocate there."""
    a = data("normal", 1 << 21)
    t = torch.from_numpy(a).cuda()
    ptr, d = cs.box_of(t)
    want = oracle.hist(a, -2.0, 2.0, 65536)
    c = torch.zeros(65539, dtype=torch.int64, device="cuda")
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        cs.cube_hist_async(ptr, d, -2.0, 2.0, 256, c.data_ptr(), s.cuda_stream)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        cs.cube_hist_async(ptr, d, -2.0, 2.0, 65536, c.data_ptr(), s.cuda_stream)
    for k in range(3):
        c.fill_(-1)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(c.cpu().numpy().astype(np.uint64), want), k
        cs.hist(t, -2.0, 2.0, 65536)
    del g
    cs.cube_release_stream(s.cuda_stream)
