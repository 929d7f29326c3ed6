"""Adaptive windows decide alike in the one-launch solve of a small system and in the
launched loop (kernel profiling on keeps to that): (nrt / nws)^(1/k) > rho_max, also
for a negative rho_max with an even k, which every window exceeds, and where
rho_max^k underflows."""
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_parity import _assert_solve_parity, dev, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_04629_amd import amg
    amg.load_library()
    return amg


@pytest.mark.parametrize("rho_max,k", [(-1.0, 2), (-0.5, 3), (1e-200, 2), (0.0, 2), (1e9, 1), (float("inf"), 2),
                                       (float("nan"), 2)])
def test_the_same_reintroductions(lib, rho_max, k):
    from oracle import oracle as O
    A = I.aniso2d(48)
    b = I.rhs(A.n, 3)
    kw = dict(method=1, tol=1e-8, maxit=200, adaptive=True, k=k, s=1, rho_max=rho_max)
    out = []
    for launched in (False, True):
        g = lib.Hierarchy(A)
        g.sparsify(1.0, first_level=2)
        assert g.grid_use() == 2
        g.profile_enable(launched)
        x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
        out.append((host(x), g.solve(dev(b), x, **kw), host(x), [g.gamma(l) for l in range(g.nlev)]))
    o = O.OracleAMG(A)
    o.sparsify([0.0, 0.0] + [1.0] * (o.nlev - 2))
    xo, ro = o.solve(b, **kw)
    for _, r, x, gammas in out:
        _assert_solve_parity(x, r, xo, ro, 1e-8)
        assert (r.reintroductions, r.restarts) == (ro.reintroductions, ro.restarts)
        assert gammas == [o.gamma(l) for l in range(o.nlev)]
    assert (ro.reintroductions > 0) == (rho_max < 1.0)
