"""The block that a closed solver leaves behind can be given back."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_kept_block_is_given_back():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    N = 512
    psi, f, g = W.flower_mms_device(N, "cuda:0")

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    s = mg.Solver(psi, N)
    want, hist = s.solve(f, g, tol=1e-9)
    s.close()
    mg.empty_cache()
    mg.empty_cache()  # nothing left: no error
    base = free()
    for _ in range(2):
        s = mg.Solver(psi, N)
        held = base - free()
        assert held >= 64 << 20
        s.close()
        assert base - free() >= 64 << 20  # kept for the next set-up
        mg.empty_cache()
        assert base - free() <= 2 << 20   # (a page of the runtime's own)
    # a live handle keeps its block
    s = mg.Solver(psi, N)
    mg.empty_cache()
    u, h = s.solve(f, g, tol=1e-9)
    assert torch.equal(u, want) and np.array_equal(h, hist)
    s.close()
