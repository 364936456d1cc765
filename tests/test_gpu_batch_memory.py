"""What a problem of a batch takes on the device."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,planes", [(256, 96), (512, 64)])
def test_problems_of_a_batch_reserve_what_they_use(N, planes):
    """Level 0's 52 planes and vectors (with a third for the coarser levels among
    them), the coarse map (16 MB: 30 planes of N = 256, 8 of 512) and the plans'
    last chunk."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    psi, f, g = W.flower_mms_device(N, "cuda:0")
    count = 8
    mg.BatchedSolver([psi] * 2, [N] * 2).close()  # (the runtime's own memory for these kernels)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    b = mg.BatchedSolver([psi] * count, [N] * count)
    torch.cuda.synchronize()
    taken = free - torch.cuda.mem_get_info()[0]
    assert taken <= count * planes * 8 * (N + 1) ** 2
    _, hists = b.solve([f] * count, [g] * count, tol=1e-9)
    assert b.last_status == 0 and len(hists) == count
    b.close()
