"""Dot products added by the kernel that needs them (at most 1,024 partials) or
by the launch that hands the scalars to the host, and the cycle's first residual
launched ahead of the host's look: solves on both sides of the edge against the
oracle, with the bars of the other solve tests (equal counts, solutions 1e-10)."""
import numpy as np
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


@pytest.mark.parametrize("N", [300, 512, 513])   # 352, 1,024 and 1,029 workgroups of a vector kernel
def test_solves_on_both_sides_of_the_edge(lib, N):
    from oracle import oracle as O
    A = I.poisson2d(N)
    g, o = lib.Hierarchy(A, setup="device", coarsening="pmis", seed=1), O.OracleAMG(A, coarsening="pmis", seed=1)
    gam = [0.0, 0.0] + [0.1] * (o.nlev - 2)
    b, x0 = I.rhs(A.n, 5), I.rhs(A.n, 6)
    for kw in (dict(), dict(adaptive=True, k=2, s=1, rho_max=0.3)):
        g.sparsify_levels(gam)
        o.sparsify(gam)
        x = dev(x0)
        r = g.solve(dev(b), x, tol=1e-8, maxit=60, **kw)
        xo, ro = o.solve(b, x0=x0, method=1, tol=1e-8, maxit=60, **kw)
        _assert_solve_parity(host(x), r, xo, ro, 1e-8)
    g.sparsify_levels(gam)
    o.sparsify(gam)
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    r = g.solve(dev(b), x, tol=1e-10, maxit=80, precision=32)
    xo, ro = o.solve(b, method=1, tol=1e-10, maxit=80)
    assert r.converged and ro.iters <= r.iters <= ro.iters + 3
    assert np.linalg.norm(host(x) - xo) <= 1e-8 * np.linalg.norm(xo)
    again = torch.zeros_like(x)
    assert g.solve(dev(b), again, tol=1e-10, maxit=80, precision=32).iters == r.iters and torch.equal(x, again)
