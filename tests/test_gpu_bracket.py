"""One rank or the median of a large box in a single read: the bracket a
sample gives, at its edges (zeros of both signs, infinities, blanks, heavily
tied values, wanted voxels lying together, ranks at either end), against a
sort of the same voxels' order keys.  Every comparison is exact."""
import math

import pytest
import torch

import paper_1111_6661_amd as cs

pytestmark = pytest.mark.gpu

N = (3 << 24) + 4097


def _fill(name, g):
    x = torch.randn(N, device="cuda", generator=g)
    nan, inf = float("nan"), float("inf")
    i = torch.arange(N, device="cuda")
    if name == "noise":
        return x
    if name == "offset":
        return x + 1000
    if name == "constant":
        return torch.full_like(x, 2.5)
    if name == "levels":          # every value held by many voxels
        return torch.round(x * 4)
    if name == "fine levels":     # several tied values in the bracket
        return torch.round(x * 300) / 8
    if name == "zeros":           # both zeros in the middle
        return torch.where(x.abs() < 0.8, x * 0, x)
    if name == "edge":            # half of the box at one side of the middle
        return x.clamp(max=0)
    if name == "infinite":
        return torch.where(x > 0.001, inf, torch.where(x < -0.001, -inf, x))
    if name == "blanks":
        return torch.where(torch.rand(N, device="cuda", generator=g) < 0.6, nan, x)
    if name == "few":             # too few valid voxels for a sample
        return torch.where(i % 90001 == 0, x, nan)
    if name == "ramp":            # the wanted voxels lie together
        return torch.sort(x).values
    if name == "period":          # a period that divides the sample's stride
        return torch.where(i % 64 == 0, 5.0, x)
    if name == "sampled":         # the sample says nothing about the rest: a miss
        j = torch.arange(1 << 18, device="cuda")
        stride = N >> 18
        x[j * stride + ((((j * 0x9E3779B1) & 0xFFFFFFFF) * stride) >> 32)] = -1000.0
        return x
    assert name == "tiny"         # denormal
    return (i % 2000003 - 1000001).int().abs().view(torch.float32)


def _sorted(x):
    """The valid voxels in the order of their keys (-0 before +0)."""
    u = x.flatten()[~x.flatten().isnan()].view(torch.int32)
    k = torch.sort(torch.where(u < 0, u ^ 0x7FFFFFFF, u)).values
    return torch.where(k < 0, k ^ 0x7FFFFFFF, k).view(torch.float32)


def _check(x, ranks):
    v = _sorted(x)
    n = v.numel()
    a, b = v[(n - 1) // 2].item(), v[n // 2].item()
    want = (a + b) / 2.0 if n % 2 == 0 else a
    for _ in range(2):
        m, nv = cs.median(x)
        assert nv == n
        assert m == want or (math.isnan(m) and math.isnan(want))
    for k in ranks(n):
        got, ref = cs.select(x, k), v[k].item()
        assert got == ref and math.copysign(1.0, got) == math.copysign(1.0, ref), k
    with pytest.raises(Exception):
        cs.select(x, n)
    for level in (0.0, 0.001, 0.37, 0.5, 1.0):
        (got,), nv = cs.quantiles(x, [level])
        h = level * (n - 1)
        j = math.floor(h)
        a, b = v[j].item(), v[min(j + 1, n - 1)].item()
        if a == b or h == j:
            want = a
        elif math.isinf(a) or math.isinf(b):
            want = math.nan if math.isinf(a) and math.isinf(b) else a if math.isinf(a) else b
        else:
            want = a + (h - j) * (b - a)
        assert nv == n and (got == want or (math.isnan(got) and math.isnan(want))), level


@pytest.mark.parametrize("name", ["noise", "offset", "constant", "levels", "fine levels", "zeros",
                                  "edge", "sampled", "infinite", "blanks", "few", "ramp",
                                  "period", "tiny"])
def test_ranks_of_a_large_box(name):
    _check(_fill(name, torch.Generator(device="cuda").manual_seed(5)),
           lambda n: (0, 1, 77, n // 1000, n // 3, (n - 1) // 2, n - 2, n - 1))


@pytest.mark.parametrize("shape,cut", [
    ((170, 600, 530), (slice(1, 169), slice(3, 590), slice(5, 528))),
    ((8000, 130, 64), (slice(None), slice(0, 129), slice(1, 62)))])
def test_ranks_of_a_cut(shape, cut):
    g = torch.Generator(device="cuda").manual_seed(3)
    box = torch.randn(shape, device="cuda", generator=g)[cut]
    box[3, 5, 7] = float("nan")
    assert box.numel() >= N - 4097
    _check(box, lambda n: (0, n // 7, n - 1))


def test_ranks_under_a_given_partition():
    g = torch.Generator(device="cuda").manual_seed(4)
    x = torch.randn(N, device="cuda", generator=g)
    for chunk in (cs.CUBE_PARTITION_STATIC, 14, 20):
        cs.cube_set_partition(chunk)
        try:
            _check(x, lambda n: (n // 5,))
        finally:
            cs.cube_set_partition(cs.CUBE_PARTITION_AUTO)


def test_no_valid_voxel_in_a_large_box():
    with pytest.raises(Exception):
        cs.median(torch.full((N,), float("nan"), device="cuda"))
