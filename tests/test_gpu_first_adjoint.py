"""The set-up builds what the adjoint runs: the first transposed cycles of a
handle take no device memory (they run inside a backward pass, where a caller
has sized its memory already)."""
import ctypes as C

import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# levels that stream (no transposed plan of their own) and float32 levels, of a
# size whose plans do not fit in what is left of a chunk: the cut positions of
# N = 4096 alone take 64 MB; 32 MB are left for graphs and the runtime
@pytest.mark.parametrize("precision", [0, 1])
def test_first_adjoint_takes_no_memory(precision):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    N = 8192
    psi, f, g = W.flower_mms_device(N, "cuda:0")
    s = mg.Solver(psi, N, precision=precision)
    u, _ = s.solve(f, g, tol=-1.0, max_cycles=2, raise_on_fail=False)
    lam = torch.empty_like(u)
    n = C.c_int32(0)
    for call in range(2):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        rc = mg._lib.lib().mgfem_adjoint(s.handle, u.data_ptr(), -1.0, 2, lam.data_ptr(), None, None, None, C.byref(n))
        assert rc == mg._lib.OK and n.value == 2
        assert free - torch.cuda.mem_get_info()[0] <= 32 << 20
    s.close()
