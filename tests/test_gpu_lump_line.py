"""Levels on either side of a third of their entries dropped, where strong
lumping turns from the lists of dropped entries to a workgroup per row: each
sparsified operator equals the oracle's bit for bit, and both sides occur."""
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_strong_lump import same_operators

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("gamma,many", [(0.01, False), (1.0, True)], ids=["lists", "workgroups"])
@pytest.mark.parametrize("make", [lambda: I.poisson3d(64), lambda: I.fv3d_lognormal(60)], ids=["poisson", "fv"])
def test_line_bitwise(make, gamma, many):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import oracle as O

    from paper_1512_04629_amd import amg
    A = make()
    g, o = amg.Hierarchy(A), O.OracleAMG(A)
    g.set_lumping("strong")
    o.set_lumping("strong")
    gam = [0.0, 0.0] + [gamma] * (o.nlev - 2)
    g.sparsify_levels(gam)
    o.sparsify(gam)
    shares = [1 - len(o.export(l, "AHAT").col) / len(o.export(l, "A").col)
              for l in range(2, o.nlev) if o.sizes(l)["n"] >= 8192]
    assert shares and any(s > 1 / 3 for s in shares) == many, shares
    same_operators(g, o)
