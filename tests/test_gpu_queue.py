"""The norm of an iterate is reduced while the next cycle's first steps run:
a solve returns the iterate whose norm met the tolerance, whatever those steps
wrote, and a profiled solve (which launches that reduction by itself) runs the
same iteration."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# fused levels (third buffer with two steps down, none with one), no cut
# sweeps, no pre-smoothing, separate kernels in both tile shapes
@pytest.mark.parametrize("N,coarsest,kw", [
    (64, 4, {}), (96, 3, {"nu1": 1, "nu2": 2}), (128, 4, {"nu1": 3, "nu2": 2}), (128, 4, {"nu1": 0, "nu2": 2}),
    (256, 4, {"eta": 0}), (768, 3, {"cycle": 2}), (1536, 3, {}), (1536, 3, {"nu1": 0, "nu2": 2}), (1536, 3, {"eta": 0}),
    (2048, 4, {}),
])
def test_steps_behind_the_norm_leave_its_iterate(N, coarsest, kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    p = W.flower_mms(N)
    s = mg.Solver(p.psi, N, coarsest_n=coarsest, **kw)
    for m in (1, 2, 3):
        u, h = s.solve(p.f, p.g, tol=-1.0, max_cycles=m)
        assert len(h) == m + 1
        us, hs = s.solve(p.f, p.g, tol=h[m] / h[0] * (1 + 1e-9), max_cycles=50)
        assert np.array_equal(hs, h) and torch.equal(u, us)
        # the norm is that of the iterate returned: F - A u from a start at u
        _, hw = s.solve(p.f, p.g, tol=-1.0, max_cycles=0, u0=u, raise_on_fail=False)
        assert abs(hw[0] - h[m]) <= 1e-10 * h[0]
        s.profile(True, repeat=2)
        up, hp = s.solve(p.f, p.g, tol=-1.0, max_cycles=m)
        s.profile(False)
        assert np.array_equal(hp, h) and torch.equal(u, up)


@pytest.mark.parametrize("N,coarsest,kw", [(64, 4, {}), (1536, 3, {}), (128, 4, {"mixed": True})])
def test_iteration_queued_before_the_first_norm(N, coarsest, kw):
    """Data whose residual is zero or not finite from the start: the zero
    vector comes back, and the next solve and adjoint are not touched."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    p = W.flower_mms(N)
    s = mg.Solver(p.psi, N, coarsest_n=coarsest, precision=mg.PREC_MIXED if kw.get("mixed") else mg.PREC_FP64)
    u, h = s.solve(p.f, p.g, tol=1e-9)
    lam = s.adjoint(u, tol=1e-9)[2]
    zero = torch.zeros_like(u)
    uz, hz = s.solve(zero, zero, tol=1e-9)
    assert len(hz) == 1 and hz[0] == 0.0 and not uz.any()
    un, hn = s.solve(zero + float("nan"), p.g, tol=1e-9, raise_on_fail=False)
    assert len(hn) == 1 and not np.isfinite(hn[0]) and not un.any()
    assert s.last_status == mg._lib.ERR_DIVERGED
    lz = s.adjoint(zero, tol=1e-9)
    assert not lz[2].any()
    u2, h2 = s.solve(p.f, p.g, tol=1e-9)
    assert np.array_equal(h, h2) and torch.equal(u, u2)
    assert torch.equal(lam, s.adjoint(u, tol=1e-9)[2])
