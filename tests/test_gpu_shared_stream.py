"""Two threads on one stream (GPU): calls of several launches that share the
stream's workspace give each thread its own cube's results, against the
oracle."""
import threading

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


@pytest.mark.parametrize("nbins,calls", [(8192, 300), (65536, 300)])
def test_two_threads_on_one_stream(cs, nbins, calls):
    n = (1 << 20) + 5
    host = [np.random.default_rng(k).standard_normal(n).astype(np.float32) * (k + 1)
            for k in range(2)]
    dev = [torch.from_numpy(h).cuda() for h in host]
    s = torch.cuda.Stream()
    outs = [torch.zeros((calls, 64), dtype=torch.uint8, device="cuda") for _ in range(2)]
    counts = [torch.zeros((calls, 2, nbins + 3), dtype=torch.int64, device="cuda")
              for _ in range(2)]
    torch.cuda.synchronize()
    gate, errors = threading.Barrier(2), []

    def work(k):
        try:
            torch.cuda.set_device(0)
            ptr, d = cs.box_of(dev[k])
            gate.wait()
            for i in range(calls):
                cs.cube_hist_async(ptr, d, -2.0, 2.0, nbins, counts[k][i, 0].data_ptr(),
                                   s.cuda_stream)
                cs.cube_stats_hist_minmax_async(ptr, d, nbins, outs[k][i].data_ptr(),
                                                counts[k][i, 1].data_ptr(), s.cuda_stream)
        except Exception as e:  # noqa: BLE001 -- shown by the assertion below
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    s.synchronize()
    assert not errors, errors
    for k in range(2):
        st = oracle.stats(host[k])
        want = (oracle.hist(host[k], -2.0, 2.0, nbins),
                oracle.hist(host[k], st.min, st.max, nbins))
        got = counts[k].cpu().numpy().astype(np.uint64)
        for j in range(2):
            wrong = [i for i in range(calls) if not np.array_equal(got[i, j], want[j])]
            assert not wrong, (k, j, len(wrong), wrong[:5])
    cs.cube_release_stream(s.cuda_stream)
