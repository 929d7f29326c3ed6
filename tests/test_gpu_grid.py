"""Small levels and small systems in one launch (grid_kernels.hip): whole PCG
solves and the cycle's small levels against the oracle at the edges of the
plan, with the bars of the other solve and V-cycle tests (equal iteration
counts, solutions 1e-10, V-cycles 1e-12 / 2e-5 in FP32), and against the same
solve launched step by step (kernel profiling on keeps to that form): the
iterates agree to the rounding of the row sums, 1e-12."""
import threading

import numpy as np
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_coarse_tail import poisson1d
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


def pair(lib, A, gamma=0.1, **kw):
    from oracle import oracle as O
    g, o = lib.Hierarchy(A, **kw), O.OracleAMG(A, **kw)
    gam = [0.0, 0.0] + [gamma] * (o.nlev - 2)
    if gamma > 0 and o.nlev > 2:
        g.sparsify_levels(gam)
        o.sparsify(gam)
    return g, o


CASES = {
    "two_levels": (lambda: I.poisson2d(9), dict(max_coarse=60)),
    "fewer_rows_than_workgroups": (lambda: I.poisson2d(5), dict(max_coarse=14)),
    "ragged_shares": (lambda: I.poisson2d(67), {}),
    "residual_exchanged": (lambda: I.random_graph_laplacian(2500), {}),
    "tail_of_many_levels": (lambda: poisson1d(1000), dict(max_coarse=2)),
    "largest_2d": (lambda: I.poisson2d(201), {}),
    "irregular_values": (lambda: I.fv3d_lognormal(23), {}),
    "cycle_only": (lambda: I.poisson3d(41), {}),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_solves_and_cycles(lib, name):
    make, kw = CASES[name]
    A = make()
    g, o = pair(lib, A, **kw)
    b, x0 = I.rhs(A.n, 5), I.rhs(A.n, 6)
    for xin in (np.zeros(A.n), x0):
        xd = dev(xin)
        g.vcycle(dev(b), xd)
        ref = o.vcycle(b, xin)
        assert np.linalg.norm(host(xd) - ref) <= 1e-12 * np.linalg.norm(ref)
        xd = dev(xin)
        r = g.solve(dev(b), xd, tol=1e-10, maxit=300)
        xo, ro = o.solve(b, x0=xin, method=1, tol=1e-10, maxit=300)
        _assert_solve_parity(host(xd), r, xo, ro, 1e-10)
        assert len(r.hist) == r.iters + 1
        # launched step by step
        xs = dev(xin)
        g.profile_enable(True)
        rs = g.solve(dev(b), xs, tol=1e-10, maxit=300)
        g.profile_enable(False)
        assert rs.iters == r.iters
        assert np.linalg.norm(host(xs) - host(xd)) <= 1e-12 * np.linalg.norm(host(xd))
        assert np.allclose(rs.hist, r.hist, rtol=0, atol=1e-9 * r.hist[0])
    # the zero guess, whatever x holds; the same bits every time
    outs = []
    for _ in range(3):
        xd = dev(x0)
        g.solve(dev(b), xd, tol=1e-10, maxit=300, zero_guess=True)
        outs.append(host(xd).tobytes())
    assert outs[0] == outs[1] == outs[2]
    x32 = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    r32 = g.solve(dev(b), x32, tol=1e-10, maxit=300, precision=32)
    xo, ro = o.solve(b, method=1, tol=1e-10, maxit=300)
    assert r32.converged and ro.iters <= r32.iters <= ro.iters + 3
    assert np.linalg.norm(host(x32) - xo) <= 1e-8 * np.linalg.norm(xo)


@pytest.mark.parametrize("gamma,rho_max,k,s", [(1.0, 0.0, 1, 1), (1.0, 0.0, 3, 2), (0.1, 0.3, 2, 1)])
def test_windows_that_reintroduce(lib, gamma, rho_max, k, s):
    """The launch ends where a window asks for a reintroduction and is resumed."""
    A = I.aniso2d(48)
    b = I.rhs(A.n, 3)
    for precision in (64, 32):
        g, o = pair(lib, A, gamma=gamma)
        kw = dict(method=1, tol=1e-8, maxit=200, adaptive=True, k=k, s=s, rho_max=rho_max)
        x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
        r = g.solve(dev(b), x, precision=precision, **kw)
        xo, ro = o.solve(b, **kw)
        assert ro.reintroductions > 0
        if precision == 64:
            _assert_solve_parity(host(x), r, xo, ro, 1e-8)
            assert (r.reintroductions, r.restarts) == (ro.reintroductions, ro.restarts)
            assert [g.gamma(l) for l in range(g.nlev)] == [o.gamma(l) for l in range(g.nlev)]
        else:
            assert r.converged and r.reintroductions > 0 and abs(r.iters - ro.iters) <= 3


def test_ends_of_a_solve(lib):
    A = I.poisson2d(40)
    g = lib.Hierarchy(A)
    b = dev(I.rhs(A.n, 2))
    x = torch.zeros_like(b)
    r = g.solve(b, x, tol=1e-14, maxit=3)                     # out of iterations
    assert r.status == -5 and r.iters == 3 and len(r.hist) == 4
    x2 = torch.zeros_like(b)
    rl = g.solve(b, x2, tol=1e-10, maxit=5000)                # more norms than a launch hands back
    x3 = torch.zeros_like(b)
    rs = g.solve(b, x3, tol=1e-10, maxit=100)
    assert rl.iters == rs.iters and torch.linalg.norm(x2 - x3) <= 1e-12 * torch.linalg.norm(x3)
    z = torch.ones_like(b)
    r = g.solve(torch.zeros_like(b), z, zero_guess=True)      # nothing to solve
    assert r.status == 0 and r.iters == 0 and not z.any()
    bad = b.clone()
    bad[7] = float("nan")
    r = g.solve(bad, torch.zeros_like(b))
    assert r.status == -6 and r.iters == 0
    x4 = torch.zeros_like(b)                                   # usable afterwards, the same bits
    g.solve(b, x4, tol=1e-10, maxit=100)
    assert torch.equal(x3, x4)


def test_cycle_in_a_captured_graph(lib):
    """The barrier's words count on from replay to replay."""
    A = I.poisson3d(24)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        g = lib.Hierarchy(A)
        b, x = dev(I.rhs(A.n, 4)), torch.zeros(A.n, dtype=torch.float64, device="cuda")
        g.vcycle(b, x)
        want = x.clone()
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            g.vcycle(b, x)
        for k in range(4):
            x.zero_()
            graph.replay()
            st.synchronize()
            assert torch.equal(x, want), k
            y = torch.zeros_like(x)
            g.vcycle(b, y)             # eager work between the replays
            st.synchronize()
            assert torch.equal(y, want), k


def test_solves_on_four_streams_at_once(lib):
    A = [I.poisson2d(64), I.random_graph_laplacian(2000), I.poisson3d(20), I.aniso2d(60)]
    jobs = []
    for k, a in enumerate(A):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            h = lib.Hierarchy(a)
            b = dev(I.rhs(a.n, k))
            x = torch.zeros_like(b)
            h.solve(b, x, tol=1e-10, maxit=200)
            st.synchronize()
            jobs.append((st, h, b, x.clone()))
    wrong = []

    def work(st, h, b, want):
        with torch.cuda.stream(st):
            for _ in range(30):
                x = torch.zeros_like(b)
                r = h.solve(b, x, tol=1e-10, maxit=200)
                st.synchronize()
                if not r.converged or not torch.equal(x, want):
                    wrong.append((h.n, r.status))

    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
