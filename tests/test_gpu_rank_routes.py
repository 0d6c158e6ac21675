"""Which way the order statistics found their ranks (GPU): the cases of the
single read and of the copies take the route that they are there for.  (Their
values are compared where the cases come from.)"""
import threading

import pytest
import torch

import paper_1111_6661_amd as cs
from tests.test_gpu_bracket import N, _fill

pytestmark = pytest.mark.gpu

HIT = ["noise", "offset", "constant", "levels", "zeros", "blanks", "ramp", "period", "tiny"]
# Half of the box in one value at one end of the bracket, or in both infinities
# around it: more than there is room to copy.
MISS = ["sampled", "few", "edge", "infinite"]


@pytest.mark.parametrize("name", HIT + MISS)
def test_single_read(name):
    x = _fill(name, torch.Generator(device="cuda").manual_seed(5))
    n = int((x == x).sum())
    want = cs.CUBE_RANK_BRACKET if name in HIT else cs.CUBE_RANK_MISSED
    known = cs.CUBE_RANK_BRACKET | cs.CUBE_RANK_MISSED
    cs.median(x)
    assert cs.cube_last_rank_route() & known == want
    cs.select(x, (n - 1) // 2)
    assert cs.cube_last_rank_route() & known == want
    cs.quantiles(x, [0.5])
    assert cs.cube_last_rank_route() & known == want
    assert cs.cube_last_quantile_reads() == 3
    cs.quantiles(x, [0.25, 0.5])          # more than one level: the passes
    assert cs.cube_last_rank_route() & known == 0


def test_one_zero_held_by_most_voxels():
    """The bracket takes both zeros, also where there is one only."""
    x = _fill("noise", torch.Generator(device="cuda").manual_seed(5))
    for zero in (0.0, -0.0):
        y = torch.where(x.abs() < 1.0, torch.full_like(x, zero), x)
        m, n = cs.median(y)
        assert m == 0.0 and n == N
        assert cs.cube_last_rank_route() == cs.CUBE_RANK_BRACKET
        got = cs.select(y, N // 2)
        assert got == 0.0 and str(got) == str(zero)
        assert cs.cube_last_rank_route() == cs.CUBE_RANK_BRACKET


def test_small_boxes_take_the_passes():
    x = torch.randn(N, device="cuda")[:(3 << 24) - 1]
    cs.median(x)
    assert cs.cube_last_rank_route() == cs.CUBE_RANK_COPIES


# The boxes of tests/test_gpu_copies.py.
@pytest.mark.parametrize("kind,route", [("spread", "COPIES"), ("crowded", "OVERFLOW"),
                                        ("many", None), ("blanks", "COPIES"),
                                        ("small", "COPIES")])
def test_copies(kind, route):
    from tests.test_gpu_copies import LEVELS
    from tests.test_gpu_copies import N as M
    g = torch.Generator(device="cuda").manual_seed(11)
    x = torch.randn(M if kind != "small" else (1 << 21) + 3, device="cuda", generator=g)
    if kind == "crowded":
        x[1 << 25:(1 << 25) + (1 << 18)] = 0.0
    elif kind == "many":
        x = torch.where(x.abs() < 0.43, torch.full_like(x, 0.125), x)
    elif kind == "blanks":
        x[::3] = float("nan")
    cs.quantiles(x, LEVELS)
    assert cs.cube_last_rank_route() == (getattr(cs, "CUBE_RANK_" + route) if route else 0)


def test_route_is_the_threads_own():
    x = torch.randn(1000, device="cuda")
    cs.median(x)
    seen = []
    t = threading.Thread(target=lambda: seen.append(cs.cube_last_rank_route()))
    t.start()
    t.join()
    assert seen == [0]
