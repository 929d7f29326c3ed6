"""Operators with few (offset, value) pairs whose slices pad too much for a SELL-64
copy stay with the LDS-staged kernel, whose sums round otherwise than the
pair-coded form's: the same bits with the compact form and without."""
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


def uneven_chain(n, every):
    """A chain with couplings 1/3; every `every`-th point is also coupled to the next
    such one by 1/7 (rows of five entries among rows of three)."""
    i = np.arange(n, dtype=np.int64)
    pairs = [(i[:-1], i[1:], 1.0 / 3.0), (i[:-every:every], i[:-every:every] + every, 1.0 / 7.0)]
    rows = np.concatenate([np.concatenate([a, b]) for a, b, _ in pairs])
    cols = np.concatenate([np.concatenate([b, a]) for a, b, _ in pairs])
    vals = np.concatenate([np.full(2 * len(a), -c) for a, _, c in pairs])
    rows, cols = np.concatenate([rows, i]), np.concatenate([cols, i])
    vals = np.concatenate([vals, np.full(n, 1.1)])
    order = np.lexsort((cols, rows))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    return I.CSR(n, rp, cols[order].astype(np.int32), vals[order])


@pytest.mark.parametrize("every,coded", [(2, False), (3, False), (64, False), (1024, True)])
def test_the_same_bits_with_and_without(lib, every, coded):
    A = uneven_chain(300_000, every)
    h, plain = lib.Hierarchy(A), lib.Hierarchy(A)
    plain.set_compact_indices(False)
    assert h.row_format(0, "A") == plain.row_format(0, "A") == ("sell" if coded else "stream")
    gen = torch.Generator(device="cuda").manual_seed(5)
    for l in range(min(2, h.nlev - 1)):
        n, nc = h.level_info(l)["n"], h.level_info(l + 1)["n"]
        b, x = (torch.rand(n, dtype=torch.float64, device="cuda", generator=gen) - 0.5 for _ in range(2))
        xc = torch.rand(nc, dtype=torch.float64, device="cuda", generator=gen) - 0.5
        for op, inp, xx, m in (("RESIDUAL", b, x, n), ("JACOBI", b, x, n), ("SPMV_A", None, x, n),
                               ("RESTRICT", x, None, nc), ("INTERPOLATE", xc, x, n)):
            out = []
            for q in (h, plain):
                y = torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")
                q.level_op(l, op, inp=inp, x=xx, out=y)
                out.append(host(y).tobytes())
            assert out[0] == out[1], (l, op)
