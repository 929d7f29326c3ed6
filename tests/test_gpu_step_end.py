"""Steps that go on after every slot has finished: the iterations left over
compute nothing, the results are bit for bit those of steps that end with the
last slot, and a right-hand side submitted afterwards starts as in a new engine."""
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_serve import lib  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("graphs", [False, True], ids=["eager", "graphs"])
@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("count", [1, 5, 16])
def test_left_over_iterations(lib, precision, graphs, count):  # noqa: F811
    A = I.poisson3d(24)
    zero = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    rhs = [torch.as_tensor(I.rhs(A.n, 50 + i)).cuda() for i in range(count)]
    rhs[-1] = zero if count == 5 else rhs[-1]      # one that is finished at once
    out = {}
    for per_step in (1, 40):                       # 40: more than any slot needs
        h = lib.Hierarchy(A)
        h.sparsify(0.01, 2)
        e = lib.Batch(h, slots=16, precision=precision, tol=1e-10, maxit=60, graphs=graphs)
        got = []
        for _ in range(3):                         # the slots are filled again after each
            slots = [e.submit(b) for b in rhs]
            left = set(slots)
            while left:
                assert e.step(per_step)
                left -= set(e.poll())
            for s in slots:
                x = torch.full((A.n,), float("nan"), dtype=torch.float64, device="cuda")
                info = e.collect(s, x)
                torch.cuda.synchronize()
                got.append((x.cpu().numpy().tobytes(), info))
        out[per_step] = got
        e.close()
        h.close()
    assert out[1] == out[40]
    assert out[1][:count] == out[1][count:2 * count] == out[1][2 * count:]
