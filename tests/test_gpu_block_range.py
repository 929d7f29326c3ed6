"""Infinities in a block cycle reach only what the arithmetic gives them: in the form
that deals a row's entries to several lanes, places past a row's end are not
multiplied.  A Poisson problem beside a clique of positive couplings, whose points
are F points without interpolation: there the cycle is two Jacobi sweeps, and with
an infinite last right-hand side entry all other points of the clique end at -inf."""
import numpy as np
import pytest

from paper_1512_04629_amd import inputs as I

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_04629_amd import amg
    amg.load_library()
    return amg


def with_clique(A, m):
    at, c = np.meshgrid(np.arange(m), np.arange(m), indexing="ij")
    v = np.where(at == c, 4.0, 1.0 / m).ravel()
    rp = np.concatenate([A.row_ptr, A.row_ptr[-1] + m * np.arange(1, m + 1)]).astype(np.int32)
    return I.CSR(A.n + m, rp, np.concatenate([A.col, A.n + c.ravel()]).astype(np.int32), np.concatenate([A.val, v]))


@pytest.mark.parametrize("m", [97, 128, 201])          # rows past a step's end, at it, past it by one
@pytest.mark.parametrize("k", [4, 8, 16])
@pytest.mark.parametrize("single", [False, True])
def test_past_a_row(lib, m, k, single):
    P = I.poisson3d(10)
    A = with_clique(P, m)
    h = lib.Hierarchy(A)
    t = torch.float32 if single else torch.float64
    gen = torch.Generator(device="cuda").manual_seed(m)
    B = torch.rand(A.n, k, dtype=t, device="cuda", generator=gen) - 0.5
    X = torch.zeros_like(B)
    h.vcycle_block(B, X)
    want = X.clone()
    assert torch.isfinite(want).all()
    B[-1, 1] = float("inf")
    X.zero_()
    h.vcycle_block(B, X)
    others = [c for c in range(k) if c != 1]
    assert torch.equal(X[:, others], want[:, others])
    assert torch.equal(X[:P.n, 1], want[:P.n, 1])
    assert torch.equal(X[P.n:-1, 1], torch.full((m - 1,), -float("inf"), dtype=t, device="cuda"))
    assert torch.isnan(X[-1, 1])
