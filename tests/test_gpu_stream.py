"""The streaming passes of the largest levels (downwards two sweeps, residual and
restriction, upwards prolongation and a sweep, over windows away from the
boundary; the fused steps or the separate kernels on the band along it) against
the separate kernels everywhere, which a profiled solve of a handle without
cut-vertex plans runs."""
import os

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# one and two levels that stream (32- and 16-row tiles), a bounding box from an
# odd column, domains that reach the sides of the grid, no cut sweeps, more
# sweeps up, a small domain (few windows)
CASES = [
    (4096, 4, lambda N: W.flower(N), {}),
    (4096, 4, lambda N: W.ellipse(N, center=(0.0517, -0.0321)), {"cycle": 2}),
    (4608, 9, lambda N: W.circle(N, radius=1.1, center=(0.1, 0.0)), {"nu2": 2, "eta": 0}),
    (4096, 8, lambda N: W.circle(N, radius=0.12, center=(0.2, 0.1)), {}),
    (1536, 3, lambda N: W.circle(N, radius=0.9), {}),
    (2048, 4, lambda N: W.flower(N), {"cycle": 3, "coarse_cycles": 2}),
    (8192, 4, lambda N: W.flower(N), {"eta": 1}),
    (1024, 4, lambda N: W.circle(N, radius=1.2, center=(0.03, 0.0)), {}),
    (1536, 3, lambda N: W.circle(N, radius=1.3), {"coarse_op": 1}),
]


def _setup(N, coarsest, psi, **kw):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_05105_amd as mg
    gen = torch.Generator(device="cuda:0").manual_seed(N)
    data = [2 * torch.rand((N + 1) ** 2, generator=gen, device="cuda:0", dtype=torch.float64) - 1 for _ in range(3)]
    if kw.pop("mixed", False):
        kw["precision"] = mg.PREC_MIXED
    separate = kw.pop("separate", False)
    if separate:
        os.environ["MGFEM_NO_CUT_GROUPS"] = "1"
    try:
        s = mg.Solver(psi(N), N, coarsest_n=coarsest, **kw)
    finally:
        os.environ.pop("MGFEM_NO_CUT_GROUPS", None)
    if separate:
        s.profile(True)
    return s, data


@pytest.mark.parametrize("N,coarsest,psi,kw", CASES)
def test_streamed_iterates(N, coarsest, psi, kw):
    """float64 iterates to 1e-10 of their largest entry on random data."""
    s, (f, g, u0) = _setup(N, coarsest, psi, **kw)

    def close(a, b, ha, hb):
        assert float((a - b).abs().max()) <= 1e-10 * float(b.abs().max())
        np.testing.assert_allclose(ha, hb, rtol=1e-9, atol=1e-12 * hb[0])

    u, h = s.solve(f, g, tol=-1.0, max_cycles=3)
    uw, hw = s.solve(f, g, tol=-1.0, max_cycles=2, u0=u0)
    sep, _ = _setup(N, coarsest, psi, separate=True, **kw)
    us, hs = sep.solve(f, g, tol=-1.0, max_cycles=3)
    uws, hws = sep.solve(f, g, tol=-1.0, max_cycles=2, u0=u0)
    close(u, us, h, hs)
    close(uw, uws, hw, hws)
    # a profiled solve of the streaming handle is the same solve
    s.profile(True)
    up, hp = s.solve(f, g, tol=-1.0, max_cycles=3)
    cycles = s.profile_read(0)["launches"]
    s.profile(False)
    close(up, u, hp, h)
    assert cycles == 3 * (kw.get("nu2", 1) + 2) + 1
    # transposed cycles run the separate kernels on such levels
    lam, lams = s.adjoint(g, tol=-1.0, max_cycles=2)[2], sep.adjoint(g, tol=-1.0, max_cycles=2)[2]
    assert float((lam - lams).abs().max()) <= 1e-10 * float(lams.abs().max())
    # the same bits again, and stopped by the tolerance instead
    u2, h2 = s.solve(f, g, tol=h[3] / h[0] * (1 + 1e-9), max_cycles=50)
    assert np.array_equal(h, h2) and torch.equal(u, u2)


@pytest.mark.parametrize("N,coarsest,psi,kw", CASES)
def test_streamed_float_cycles_keep_their_bits(N, coarsest, psi, kw):
    """float32 cycles do not depend on which kernel computed a node."""
    s, (f, g, _) = _setup(N, coarsest, psi, mixed=True, **kw)
    u, h = s.solve(f, g, tol=-1.0, max_cycles=3)
    s.profile(True)
    us, hs = s.solve(f, g, tol=-1.0, max_cycles=3)
    s.profile(False)
    assert np.array_equal(h, hs) and torch.equal(u, us)


@pytest.mark.parametrize("N,coarsest,psi,kw,streams", [
    (2048, 4, lambda N: W.flower(N), {}, True),
    (1536, 3, lambda N: W.circle(N, radius=1.1), {"cycle": 2}, True),
    (512, 4, lambda N: W.flower(N), {}, False),
    (2048, 4, lambda N: W.flower(N), {"nu2": 2}, False),
])
def test_profiled_passes_are_those_of_the_solve(N, coarsest, psi, kw, streams):
    """One downward pass per cycle and one behind the last, one upward pass per
    cycle, timed where they run: the solve's bits stay, repeated launches too."""
    s, (f, g, _) = _setup(N, coarsest, psi, **kw)
    u, h = s.solve(f, g, tol=-1.0, max_cycles=3)
    for repeat in (1, 3):
        s.profile(True, repeat=repeat)
        up, hp = s.solve(f, g, tol=-1.0, max_cycles=3)
        down, upward = s.profile_read(2), s.profile_read(3)
        s.profile(False)
        assert np.array_equal(h, hp) and torch.equal(u, up)
        assert down["launches"] == (4 if streams else 0) and upward["launches"] == (3 if streams else 0)
        n = s.level_counts(0)["n_active"]
        if streams:  # the first pass starts from zero and does not read its iterate
            assert 0 < down["alg_bytes"] <= (3 * 26 + 18) * n and down["total_ms"] > 0.0
            assert 0 < upward["alg_bytes"] <= 3 * 26 * n and upward["total_ms"] > 0.0


def test_streamed_float_cycles_from_an_odd_column():
    """float32 windows start at an even column and row, the active nodes here at odd ones."""
    N = 4608
    s, (f, g, _) = _setup(N, 9, lambda N: W.circle(N, radius=0.8995), mixed=True)
    import paper_2505_05105_amd as mg
    on = (s.export(mg._lib.EXPORT_NODE_FLAGS) > 0).view(N + 1, N + 1)
    assert int(on.any(0).nonzero()[0]) % 2 == 1 and int(on.any(1).nonzero()[0]) % 2 == 1
    u, h = s.solve(f, g, tol=-1.0, max_cycles=2)
    s.profile(True)
    us, hs = s.solve(f, g, tol=-1.0, max_cycles=2)
    s.profile(False)
    assert np.array_equal(h, hs) and torch.equal(u, us)


@pytest.mark.parametrize("kw", [{"mixed": True}, {"nu1": 4, "nu2": 3}, {"mixed": True, "inner_cycles": 16, "nu2": 2}])
def test_profiled_iterations_are_captured(kw, capfd):
    """However many launches an iteration times, it is still replayed as a graph
    (a capture that fails is reported, and ends the handle's replays)."""
    s, (f, g, _) = _setup(256, 4, lambda N: W.flower(N), **kw)
    s.profile(True, repeat=2)
    s.solve(f, g, tol=-1.0, max_cycles=3)
    n = s.profile_read(1 if kw.get("mixed") else 0)["launches"]
    per_cycle = s.params.nu1 + s.params.nu2
    assert n == (3 * s.params.inner_cycles * per_cycle if kw.get("mixed") else 3 * per_cycle + 1)
    s.close()
    assert "graph capture" not in capfd.readouterr().err
