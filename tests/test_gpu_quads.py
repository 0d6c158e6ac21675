"""Projection maps by quads of pixels: the edges of rows, quads, wavefront
shares and slices, on aligned and unaligned images, against the oracle."""
import numpy as np
import pytest

from tests.test_gpu_project import compare

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    import paper_1111_6661_amd as cs
    assert torch.cuda.is_available()
    cs.load()
    return cs


# (nx, ny, nz, x0, pitch): rows under a quad, of one quad, ragged; whole images
# as one row; 64 quads and one more; slices; the shares of 4, 5 and more quads
# per lane, whole and cut images, the last wavefront overlapping its neighbour;
# 16 quads per lane and past it.
CASES = [(1, 5, 9, 0, 1), (3, 7, 33, 1, 8), (4, 9, 5, 3, 9), (5, 9, 70, 0, 5), (7, 1, 40, 2, 16),
         (256, 1, 3, 0, 256), (257, 3, 64, 1, 259), (61, 47, 200, 5, 512), (1000, 787, 2, 0, 1000),
         (1001, 787, 5, 3, 1024), (1024, 1024, 3, 0, 1024), (1024, 1025, 6, 1, 1030),
         (2047, 700, 2, 0, 2047), (2041, 513, 7, 5, 2048), (4099, 1100, 2, 0, 4099),
         (4096, 1040, 2, 0, 4096)]


@pytest.mark.parametrize("case", CASES, ids=str)
def test_quads(cs, case):
    nx, ny, nz, x0, pitch = case
    rng = np.random.default_rng(sum(case))
    extra = 0 if pitch == nx else 1          # cut images: rows and planes apart
    a = rng.standard_normal((nz, ny + extra, pitch)).astype(np.float32)
    a[rng.random(a.shape) < 0.05] = np.nan
    a[:, ny // 2, x0] = np.nan
    t = torch.from_numpy(a).cuda()
    v, h = t[:, extra:, x0:x0 + nx], a[:, extra:, x0:x0 + nx]
    guard = torch.full((ny * nx + 8,), 7.0, dtype=torch.float32, device="cuda")
    ptr, d = cs.box_of(v)
    compare(cs.project(v), np.ascontiguousarray(h), f"{case}")
    cs.cube_project(ptr, d, mip=guard[4:].data_ptr())       # one map, at a 16-byte offset
    g = guard.cpu().numpy()
    assert (g[:4] == 7.0).all() and (g[4 + nx * ny:] == 7.0).all()
    want = cs.project(v)[0].cpu().numpy().reshape(-1)
    assert np.array_equal(g[4:4 + nx * ny].view(np.uint32), want.view(np.uint32))
