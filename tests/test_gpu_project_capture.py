"""Projections captured into HIP graphs (GPU): on a stream without memory for
the slices' partials, and on one that makes room for a larger projection
afterwards; every replay against the oracle."""
import numpy as np
import pytest

from tests.test_gpu_project import compare, cube_of

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def cs():
    import paper_1111_6661_amd as cs
    assert torch.cuda.is_available()
    cs.load()
    return cs


def maps(ny, nx):
    return (torch.empty((ny, nx), dtype=torch.float32, device="cuda"),
            torch.empty((ny, nx), dtype=torch.float64, device="cuda"),
            torch.empty((ny, nx), dtype=torch.int32, device="cuda"))


def queue(cs, v, out, s):
    ptr, d = cs.box_of(v)
    cs.cube_project(ptr, d, out[0].data_ptr(), out[1].data_ptr(), out[2].data_ptr(),
                    s.cuda_stream)


def replays(cs, g, v, out, host, other):
    """Three replays, each over outputs overwritten meanwhile and with eager
    work between them."""
    for k in range(3):
        for o in out:
            o.fill_(7)
        cs.project(other)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        compare(out, host, f"replay {k}")


# Slices where there is room for their partials: an unaligned cut, and a whole image.
@pytest.mark.parametrize("warm", [False, True])
@pytest.mark.parametrize("cut", [True, False])
def test_captured_projection(cs, cut, warm):
    big = cube_of((128, 260, 520), 21)
    v = big[:, 3:259, 5:517] if cut else big[:, :256].contiguous()
    host = np.ascontiguousarray(v.cpu().numpy())
    out = maps(*v.shape[1:])
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    if warm:
        queue(cs, v, out, s)
        s.synchronize()
        compare(out, host, "eager")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        queue(cs, v, out, s)
    replays(cs, g, v, out, host, v)
    del g


def test_a_captured_projection_outlives_a_larger_one(cs):
    """The graph's partials stay where they are when a later projection on the
    stream needs more of them."""
    big = cube_of((256, 500, 517), 5)
    v = big[:, :256, :256].contiguous()
    host, host_big = v.cpu().numpy(), big.cpu().numpy()
    out, out_big = maps(256, 256), maps(500, 517)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    queue(cs, v, out, s)
    s.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        queue(cs, v, out, s)
    queue(cs, big, out_big, s)
    s.synchronize()
    compare(out_big, host_big, "larger")
    replays(cs, g, v, out, host, big)
    del g
