"""The pair-coded form of operators with few distinct (offset, value) pairs per
block of rows: a lossless storage form, so every row operation gives bit for bit
what the 32-bit SELL-64 copy or the LDS-staged kernel gives (compact indices
off), and the oracle's values within the row bar 1e-13 (|M||v| + |u|)."""
import numpy as np
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_parity import dev, host

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_04629_amd import amg
    amg.load_library()
    return amg


def with_values(A, kinds):
    """A with its off-diagonal couplings scaled by one of `kinds` factors, the
    factor of an edge chosen by its ends (symmetric; the diagonal stays)."""
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    lo, hi = np.minimum(rows, A.col).astype(np.int64), np.maximum(rows, A.col).astype(np.int64)
    f = 1.0 - ((lo * 31 + hi * 17) % kinds) / (4.0 * kinds)
    v = np.where(rows == A.col, A.val, A.val * f)
    return I.CSR(A.n, A.row_ptr, A.col, v)


CASES = {
    # ragged last block (rows not a multiple of 256), 7 pairs a block
    "poisson3d_67": (lambda: I.poisson3d(67), True),
    # 9-point rows; interpolation of one word
    "aniso2d_701": (lambda: I.aniso2d(701), True),
    # interpolation large enough for the coded form
    "poisson3d_75": (lambda: I.poisson3d(75), True),
    # near the limit of a table: 30 values on 7 offsets, about 180 pairs a block
    "many_pairs": (lambda: with_values(I.poisson3d(66), 30), True),
    # past it: the SELL-64 copy stays
    "too_many_pairs": (lambda: with_values(I.poisson3d(66), 401), False),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_coded_rows_bitwise(lib, name):
    make, coded = CASES[name]
    A = make()
    h = lib.Hierarchy(A)
    plain = lib.Hierarchy(A)
    before = plain.device_bytes()
    plain.set_compact_indices(False)
    gen = torch.Generator(device="cuda").manual_seed(7)
    if coded:
        assert h.index_width(0, "A") == 1 and h.row_format(0, "A") == "sell"
        assert before < plain.device_bytes()
    for l in range(min(3, h.nlev - 1)):
        n, nc = h.level_info(l)["n"], h.level_info(l + 1)["n"]
        b, x = (torch.rand(n, dtype=torch.float64, device="cuda", generator=gen) - 0.5 for _ in range(2))
        xc = torch.rand(nc, dtype=torch.float64, device="cuda", generator=gen) - 0.5
        for op, inp, xx, m in (("RESIDUAL", b, x, n), ("JACOBI", b, x, n), ("SPMV_A", None, x, n),
                               ("RESTRICT", x, None, nc), ("INTERPOLATE", xc, x, n)):
            want = torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")
            plain.level_op(l, op, inp=inp, x=xx, out=want)
            for _ in range(2):          # both directions over the blocks
                got = torch.full((m,), float("nan"), dtype=torch.float64, device="cuda")
                h.level_op(l, op, inp=inp, x=xx, out=got)
                assert host(got).tobytes() == host(want).tobytes(), (l, op)
    b = dev(I.rhs(A.n, 4))
    for precision in (64, 32):
        out = []
        for q in (h, plain):
            x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
            r = q.solve(b, x, tol=1e-10, maxit=60, adaptive=precision == 64, precision=precision)
            out.append((r.iters, host(x).tobytes(), r.hist.tobytes()))
        assert out[0] == out[1], precision


def test_values_out_of_range_reach_only_their_rows(lib):
    """A column that holds an infinity or a NaN spoils the rows that have it and no
    others: padded slots are not summed."""
    A = I.poisson3d(67)
    h = lib.Hierarchy(A)
    assert h.index_width(0, "A") == 1
    rows = np.repeat(np.arange(A.n), np.diff(A.row_ptr))
    for at, bad in ((0, np.inf), (A.n - 1, np.nan), (A.n // 2, -np.inf)):
        x = np.ones(A.n)
        x[at] = bad
        y = torch.zeros(A.n, dtype=torch.float64, device="cuda")
        h.level_op(0, "SPMV_A", x=dev(x), out=y)
        touched = np.zeros(A.n, bool)
        touched[rows[A.col == at]] = True
        assert np.array_equal(~np.isfinite(host(y)), touched)
