"""The extra smoothing in groups of one wave against the list smoother (one
launch per colour phase, MGFEM_NO_CUT_GROUPS=1), where a group's closure ends:
along rows, columns and diagonals, at the sides of the grid, and with more
closure nodes than lanes (tiles split, or the groups of four waves)."""
import os

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _crowded(N):
    x, y = W.grid_xy(N)
    return np.cos(np.pi * N / 8 * (x + 0.013)) * np.cos(np.pi * N / 8 * (y - 0.007)) - 0.35


@pytest.mark.parametrize("N,psi,eta", [
    (64, lambda N: W.circle(N, radius=0.6), 1), (96, lambda N: W.flower(N), 4),
    (160, lambda N: W.ellipse(N, center=(0.05, -0.03)), 3), (320, lambda N: W.circle(N, radius=1.1), 4),
    (64, _crowded, 4), (64, lambda N: W.flower(N), 7),
])
@pytest.mark.parametrize("reverse", [False, True])
def test_groups_match_the_list_smoother(N, psi, eta, reverse):
    """Two steps on random data, to 1e-12 of the largest entry (the two differ
    in the rounding of 2 (eta + 1) sweeps)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    psi = psi(N)
    kw = {"eta": eta, "coarsest_n": 5 if N % 5 == 0 else 4 if N % 3 else 3}
    s = mg.Solver(psi, N, **kw)
    os.environ["MGFEM_NO_CUT_GROUPS"] = "1"
    try:
        ref = mg.Solver(psi, N, **kw)
    finally:
        del os.environ["MGFEM_NO_CUT_GROUPS"]
    gen = torch.Generator(device="cuda:0").manual_seed(N + eta)
    on = s.export(mg._lib.EXPORT_NODE_FLAGS) > 0
    x, b = (torch.rand((N + 1) ** 2, generator=gen, device="cuda:0", dtype=torch.float64) - 0.5 for _ in range(2))
    x, b = x * on, b * on
    a = s.smooth(0, x.clone(), b, steps=2, reverse=reverse)
    r = ref.smooth(0, x.clone(), b, steps=2, reverse=reverse)
    assert float((a - r).abs().max()) <= 1e-12 * float(r.abs().max())
