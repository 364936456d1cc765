"""The one-pass misfit (J and dJ/du) at the edges of its 256 x 8-node blocks,
against the assembled mass matrix of the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import assembly as oasm

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# one block, a block and one node, blocks that end on the grid's side, a domain
# over the sides of the box
@pytest.mark.parametrize("N,coarsest,psi", [
    (6, 3, lambda N: W.circle(N, radius=0.8)),
    (8, 4, lambda N: W.circle(N, radius=0.8)),
    (256, 4, lambda N: W.flower(N)),
    (320, 5, lambda N: W.circle(N, radius=1.1)),
    (512, 4, lambda N: W.ellipse(N)),
])
def test_misfit_at_block_edges(N, coarsest, psi):
    """Rounding only: sums of 9 terms a row (1e-13 of the largest entry), J to
    1e-12 as in the parity test's sums; values at inactive nodes (NaN here) have
    no share; a gradient written over u gives the same."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    psi = psi(N)
    d = oasm.assemble(psi, N)
    rng = np.random.default_rng(N)
    u, ut = rng.uniform(-1, 1, d.n), rng.uniform(-1, 1, d.n)
    e = np.where(d.active, u - ut, 0.0)
    Me = d.M @ e
    s = mg.Solver(psi, N, coarsest_n=coarsest)
    ud = torch.tensor(np.where(d.active, u, np.nan), device="cuda:0")
    utd = torch.tensor(ut, device="cuda:0")
    J, g = s.misfit(ud, utd)
    assert J == pytest.approx(0.5 * e @ Me, rel=1e-12)
    assert np.abs(g.cpu().numpy() - Me).max() <= 1e-13 * np.abs(Me).max()
    import ctypes as C
    from paper_2505_05105_amd import _lib
    J2 = C.c_double(0.0)
    _lib.check(_lib.lib().mgfem_misfit(s.handle, ud.data_ptr(), utd.data_ptr(), C.byref(J2), ud.data_ptr()), s.handle)
    assert J2.value == J and torch.equal(ud, g)
