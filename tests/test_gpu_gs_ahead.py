"""Gauss-Seidel chains whose staging waves subtract a row's leading terms and
own contiguous shares of a strip: the smallest grid whose second level takes two
such waves of 16 lanes (1,024 chunks or more, rows above 8), chunks of rows that
straddle the shares of four, one of 16 lanes on rows of up to 8, and the chunk
lengths on either side of the line.  Each sweep does the oracle's operations on
a row in the oracle's order, so the bar is equality of every bit."""
import numpy as np
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_parity import dev, host
from .test_gpu_relax import lib, pair  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,block", [(53, 64), (53, 16), (41, 32), (41, 31), (30, 64), (30, 200)],
                         ids=["two_waves_16", "blocks_in_a_chunk", "chunk_32", "chunk_31", "four_waves_64",
                              "many_strips"])
def test_terms_ahead_bitwise(lib, n, block):  # noqa: F811
    A = I.poisson3d(n)
    g, o = pair(A, block)
    rng = np.random.default_rng(23)
    for l in range(o.nlev - 1):
        m = o.sizes(l)["n"]
        b, x = rng.standard_normal(m), rng.standard_normal(m)
        b[m // 3] = 0.0
        for op, code in (("GS_FORWARD", 7), ("GS_BACKWARD", 8)):
            out = torch.zeros(m, dtype=torch.float64, device="cuda")
            g.level_op(l, op, dev(b), dev(x), out)
            assert host(out).tobytes() == o.level_op(l, code, b, x, m).tobytes(), (l, op)
