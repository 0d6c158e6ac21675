"""Packed rows (cube_rows.h) on the GPU: every pass over boxes of short rows,
against the oracle, at the edges of the lanes, the tiles and the alignments.

Counts, extrema and order statistics must be exact; mean and std meet the
repository's rule for moments (tests/parity.py).
"""
import numpy as np
import pytest

import oracle
from tests.parity import mean_ok, std_ok

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    import paper_1111_6661_amd as cs
    assert torch.cuda.is_available()
    cs.load()
    return cs


def box(nx, ny, nz, x0, pitch, seed):
    """(device view, host copy) of a box at x0 in rows of `pitch` voxels."""
    rng = np.random.default_rng(seed)
    a = rng.standard_normal((nz + 1, ny + 2, pitch)).astype(np.float32)
    a[rng.random(a.shape) < 0.01] = np.nan
    a[0, 0, x0] = np.float32(7.5)
    t = torch.from_numpy(a).cuda()
    v = t[:nz, 1:1 + ny, x0:x0 + nx]
    return v, np.ascontiguousarray(a[:nz, 1:1 + ny, x0:x0 + nx])


# (nx, ny, nz, x0, pitch): one vector; ragged; every alignment on even and odd
# pitches; column groups of 1, 2 and 4; the last packed length of 256-, 512-
# and 1024-thread blocks and the first that is not; one row a plane, one plane.
CASES = [(4, 9, 11, 1, 9), (5, 300, 3, 2, 8), (61, 47, 20, 1, 512), (61, 47, 20, 2, 511),
         (61, 47, 20, 3, 512), (63, 5, 700, 0, 64), (257, 33, 9, 3, 1024), (340, 40, 7, 1, 344),
         (1187, 91, 3, 341, 2048), (1187, 91, 3, 2, 2047), (2048, 1, 50, 1, 2052),
         (4096, 6, 5, 3, 4100), (4097, 6, 5, 3, 4101), (4100, 12, 1, 0, 4104),
         (8192, 5, 4, 1, 8196), (16384, 3, 4, 2, 16388), (16388, 3, 4, 2, 16392),
         (100, 1200, 14, 5, 108)]


@pytest.mark.parametrize("case", CASES, ids=str)
@pytest.mark.parametrize("chunk", [0, 13])
def test_rows_all_passes(cs, case, chunk):
    v, h = box(*case, seed=sum(case))
    ref = oracle.stats(h)
    lo, hi, nb = -1.5, 2.0, 100
    want = oracle.hist(h, lo, hi, nb)
    ptr, d = cs.box_of(v)
    prev = cs.cube_set_partition(chunk)
    try:
        for st in (cs.stats(v), cs.stats_hist(v, lo, hi, nb)[0], cs.stats_hist_minmax(v, nb)[0]):
            assert (st.n_valid, st.n_nan, st.min, st.max) == (ref.n_valid, ref.n_nan, ref.min,
                                                              ref.max)
            assert mean_ok(st.mean, ref) and std_ok(st.std, ref), (st, ref)
        assert np.array_equal(cs.stats_hist(v, lo, hi, nb)[1], want)
        assert np.array_equal(cs.hist(v, lo, hi, nb), want)
        assert np.array_equal(cs.hist(v, lo, hi, 40000), oracle.hist(h, lo, hi, 40000))
        assert np.array_equal(cs.stats_hist_minmax(v, nb)[1],
                              oracle.hist(h, float(ref.min), float(ref.max), nb))
        rank = ref.n_valid // 3
        assert cs.select(v, rank) == np.float32(oracle.select(h, rank))
        assert cs.median(v)[0] == oracle.median(h)
        q = [0.0, 0.01, 0.5, 0.77, 1.0]
        assert np.array_equal(cs.quantiles(v, q)[0], oracle.quantiles(h, q))
    finally:
        cs.cube_set_partition(prev)


@pytest.mark.parametrize("threads", [256, 512, 1024])
def test_rows_in_a_batch(cs, threads):
    boxes = [box(*c, seed=sum(c)) for c in CASES]
    nb = 64
    outs = torch.zeros((len(boxes), 64), dtype=torch.uint8, device="cuda")
    cnt = torch.zeros((len(boxes), nb + 3), dtype=torch.int64, device="cuda")
    kinds = [cs.CUBE_Q_MINMAX, cs.CUBE_Q_FUSED, cs.CUBE_Q_STATS]
    qs = []
    for i, (v, _) in enumerate(boxes):
        ptr, d = cs.box_of(v)
        qs.append(cs.make_query(ptr, d, kinds[i % 3], nb, -1.0, 1.0, outs[i].data_ptr(),
                                cnt[i].data_ptr()))
    b = cs.Batch(tile_voxels=4096, threads=threads)
    b.enqueue(qs)
    b.check()
    for i, (v, h) in enumerate(boxes):
        st, ref = cs.Stats.from_bytes(bytes(outs[i].cpu().numpy())), oracle.stats(h)
        assert (st.n_valid, st.n_nan, st.min, st.max) == (ref.n_valid, ref.n_nan, ref.min, ref.max)
        assert mean_ok(st.mean, ref) and std_ok(st.std, ref), (i, st, ref)
        if i % 3 != 2:
            lo, hi = (float(ref.min), float(ref.max)) if i % 3 == 0 else (-1.0, 1.0)
            assert np.array_equal(cnt[i].cpu().numpy().astype(np.uint64),
                                  oracle.hist(h, lo, hi, nb)), i
