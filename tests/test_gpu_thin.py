"""Statistics and order statistics of boxes whose rows are too short for a float4 (GPU): the
spectrum of a pixel, columns of two and three, against the oracle."""
import numpy as np
import pytest

import oracle
from tests.parity import assert_counts_match, assert_stats_match

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("shape", [(1, 1, 1), (7, 1, 1), (1000, 1, 1), (5000, 1, 1), (1024, 5, 1),
                                   (200, 200, 2), (4000, 3, 3), (1, 1000, 1), (1, 70000, 3)], ids=str)
def test_thin_boxes(shape):
    import paper_1111_6661_amd as cs
    cs.load()
    g = torch.Generator(device="cuda").manual_seed(sum(shape))
    p = torch.randn(tuple(n + 2 for n in shape), device="cuda", generator=g)
    p[torch.rand(p.shape, device="cuda", generator=g) < 0.05] = float("nan")
    p[1, 1, 1] = 0.5
    v = p[1:-1, 1:-1, 1:-1]
    host = np.ascontiguousarray(v.cpu().numpy())
    valid = np.sort(host[~np.isnan(host)])
    n = valid.size
    assert cs.median(v) == ((float(valid[(n - 1) // 2]) + float(valid[n // 2])) / 2, n)
    st, counts = cs.stats_hist(v, -2.0, 2.0, 100)
    assert_stats_match(st, oracle.stats(host), str(shape))
    assert_counts_match(counts, oracle.hist(host, -2.0, 2.0, 100), str(shape))
    for k in (0, n // 3, n - 1):
        assert cs.select(v, k) == valid[k]
    levels = [i / 63 for i in range(64)]
    for lv in (levels, levels[5:9], [0.37]):
        got, nv = cs.quantiles(v, lv)
        assert nv == n
        assert np.array_equal(got.view(np.uint64), oracle.quantiles(host, lv).view(np.uint64))
