"""Interpolation from the pair-coded form has the bits of the LDS-staged kernel it
stands for also where the rows of P would fit a SELL-64 copy, whose sums round
differently: C points first, then F points (rows of one and of two entries, not
mixed), weights 1/3 and 2/3."""
import numpy as np
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_parity import host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_04629_amd import amg
    amg.load_library()
    return amg


def two_colours(m):
    """A chain of 2 m + 1 points coupled by 1 and 2 in turn, its even points first."""
    n = 2 * m + 1
    at = np.empty(n, np.int64)
    at[0::2], at[1::2] = np.arange(m + 1), np.arange(m + 1, n)
    c = np.where(np.arange(n + 1) % 2 == 0, 2.0, 1.0)          # coupling of points g - 1 and g
    rows, cols, vals = [at], [at], [c[:-1] + c[1:]]
    for a, b in ((at[:-1], at[1:]), (at[1:], at[:-1])):
        rows.append(a)
        cols.append(b)
        vals.append(-c[1:-1])
    rows, cols, vals = (np.concatenate(v) for v in (rows, cols, vals))
    order = np.lexsort((cols, rows))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    return I.CSR(n, rp, cols[order].astype(np.int32), vals[order])


def test_switched_off_the_same_bits(lib):
    A = two_colours(400_000)
    h = lib.Hierarchy(A)
    assert h.index_width(0, "P") == 1 and h.row_format(0, "P") == "sell"
    n, nc = h.level_info(0)["n"], h.level_info(1)["n"]
    assert nc == 400_001
    gen = torch.Generator(device="cuda").manual_seed(3)
    x = torch.rand(n, dtype=torch.float64, device="cuda", generator=gen) - 0.5
    xc = torch.rand(nc, dtype=torch.float64, device="cuda", generator=gen) - 0.5

    def interpolate():
        y = torch.full((n,), float("nan"), dtype=torch.float64, device="cuda")
        h.level_op(0, "INTERPOLATE", inp=xc, x=x, out=y)
        return host(y).tobytes()

    want = interpolate()
    h.set_compact_indices(False)
    assert h.row_format(0, "P") == "stream"
    assert interpolate() == want
    h.set_compact_indices(True)
    assert h.index_width(0, "P") == 1 and interpolate() == want
