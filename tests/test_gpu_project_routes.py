"""Projection maps on both sides of the line between one pixel and one quad of
pixels per lane, and of those between one and more slices (GPU), against the
oracle; the quads' edges with channels enough that they are quads."""
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


def check(cs, nx, ny, nz, x0, pitch, what):
    extra = 0 if pitch == nx else 1          # cut images: rows and planes apart
    g = torch.Generator(device="cuda").manual_seed(nx + ny + nz)
    t = torch.randn((nz, ny + extra, pitch), device="cuda", generator=g)
    t[torch.rand(t.shape, device="cuda", generator=g) < 0.05] = float("nan")
    t[:, ny // 2, x0 + nx // 2] = float("nan")
    v = t[:, extra:, x0:x0 + nx]
    compare(cs.project(v), np.ascontiguousarray(v.cpu().numpy()), what)


ROUTES = [(64, 64, 39), (64, 64, 40), (64, 64, 4608), (64, 64, 4609), (256, 256, 288),
          (256, 256, 289), (450, 450, 93), (450, 450, 94), (450, 450, 96), (550, 550, 256), (550, 550, 257),
          (640, 640, 16), (640, 640, 17), (941, 937, 21), (941, 937, 22)]


@pytest.mark.parametrize("shape", ROUTES, ids=str)
@pytest.mark.parametrize("cut", [0, 1])
def test_routes(cs, shape, cut):
    nx, ny, nz = shape
    check(cs, nx, ny, nz, 3 * cut, nx + 5 * cut, f"{shape} {cut}")


# (nx, ny, x0, pitch): rows of one quad, ragged ones, whole images, a last
# wavefront that overlaps its neighbour, 4, 5 and 16 quads per lane.
EDGES = [(4, 9, 3, 9), (5, 9, 0, 5), (7, 1, 2, 16), (256, 1, 0, 256), (257, 3, 1, 259),
         (61, 47, 5, 512), (1000, 787, 0, 1000), (1001, 787, 3, 1024), (1024, 1024, 0, 1024),
         (1024, 1025, 1, 1030), (2047, 700, 0, 2047), (2041, 513, 5, 2048),
         (4099, 1100, 0, 4099), (4096, 1040, 0, 4096)]


@pytest.mark.parametrize("edge", EDGES, ids=str)
def test_quads_at_their_edges(cs, edge):
    nx, ny, x0, pitch = edge
    waves = ((nx + 3) // 4 * ny + 63) // 64
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    check(cs, nx, ny, 288 * cus // waves + 3, x0, pitch, f"{edge}")
