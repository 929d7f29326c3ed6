"""Strong-neighbour lumping by the lists of dropped entries (levels of at least
8,192 rows) with the rows of many dropped entries, and those longer than a
wave's stage, given a workgroup: every sparsified operator equals the oracle's
bit for bit, as in the other strong-lumping tests."""
import numpy as np
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_product import csr
from .test_gpu_strong_lump import same_operators

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def grid_with_hub(N, links):
    """A 3D grid with points spread over it weakly coupled to a hub, which depends
    on a partner: the hub's coarse row is as long as it has links."""
    P = I.poisson3d(N)
    i, j = np.repeat(np.arange(P.n), np.diff(P.row_ptr)), P.col
    up, k = i < j, np.arange(links) * (P.n // links)
    return csr(np.r_[i[up], k, P.n], np.r_[j[up], np.full(links, P.n), P.n + 1],
               np.r_[-P.val[up], np.full(links, 2.0**-10), [1000.0]], P.n + 2)


CASES = {   # name: matrix, drop tolerance, whether rows are to be found on both sides of 32 dropped entries
    "few_dropped": (lambda: I.poisson3d(52), 0.05, False),
    "both_forms": (lambda: I.poisson3d(60), 0.2, True),
    "nearly_all_dropped": (lambda: I.poisson3d(34), 1.0, False),
    "irregular_rows": (lambda: I.random_graph_laplacian(30000, degree=2), 0.1, False),
    "one_long_row": (lambda: grid_with_hub(40, 300), 0.2, False),   # longer than the stage, without drops of its own
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_lists_bitwise(name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle as O

    from paper_1512_04629_amd import amg
    make, gamma, both = CASES[name]
    A = make()
    g, o = amg.Hierarchy(A, setup="device", coarsening="pmis", seed=3), O.OracleAMG(A, coarsening="pmis", seed=3)
    g.set_lumping("strong")
    o.set_lumping("strong")
    gam = [0.0] + [gamma] * (o.nlev - 1)
    g.sparsify_levels(gam)
    o.sparsify(gam)
    listed = [l for l in range(1, o.nlev) if o.sizes(l)["n"] >= 8192]
    assert listed
    drops = np.concatenate([np.diff(o.export(l, "A").row_ptr) - np.diff(o.export(l, "AHAT").row_ptr) for l in listed])
    assert (drops > 0).any() and (drops <= 32).any()
    assert (drops > 32).any() or not both
    same_operators(g, o)
