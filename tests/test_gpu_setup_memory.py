"""The first chunk of a released handle serves the next set-up of its size: what
that one computes depends neither on what the chunk held nor on the stream or
thread, and at most one block per device stays behind."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _solve(mg, psi, f, g, N, **kw):
    s = mg.Solver(psi, N, **kw)
    u, h = s.solve(f, g, tol=1e-9)
    s.close()
    return u, h


# below and above the smallest block that is kept, and float cycles
@pytest.mark.parametrize("N,kw", [(128, {}), (256, {}), (512, {}), (512, {"precision": 1})])
def test_reused_block_gives_the_same_solve(N, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    psi, f, g = W.flower_mms_device(N, "cuda:0")
    want, hist = _solve(mg, psi, f, g, N, **kw)
    torch.cuda.synchronize()
    for move in (0.05, -0.05):
        _solve(mg, psi + move, f, g, N, **kw)  # leaves another geometry's arrays in the block
        torch.cuda.synchronize()
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            u, h = _solve(mg, psi, f, g, N, **kw)
        stream.synchronize()
        assert torch.equal(u, want) and np.array_equal(h, hist)


def test_handles_in_threads_and_sizes_in_turn():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    data = {N: W.flower_mms_device(N, "cuda:0") for N in (256, 512)}
    want = {N: _solve(mg, *data[N], N) for N in data}
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    bad = []

    def work(sizes):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for N in sizes:
                u, h = _solve(mg, *data[N], N)
                stream.synchronize()
                if not (torch.equal(u, want[N][0]) and np.array_equal(h, want[N][1])):
                    bad.append(N)

    threads = [threading.Thread(target=work, args=(s,)) for s in ((256, 256, 512, 256), (512, 256, 512, 512))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    # one block, of either size (0.25 GB at N = 512), and what torch's own
    # allocator took meanwhile
    assert free0 - torch.cuda.mem_get_info()[0] <= 512 << 20
