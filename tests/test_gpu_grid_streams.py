"""Launches whose workgroups wait for each other go to no more streams than can
have them on the device at the same time; handles of further streams are launched
step by step, with the same result to rounding (1e-10, the bar of the solves)."""
import gc

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


def test_streams_beyond_the_device(lib):
    gc.collect()
    A = I.poisson2d(40)
    b = I.rhs(A.n, 5)
    streams = [torch.cuda.Stream() for _ in range(16)]

    def on(st):
        with torch.cuda.stream(st):
            return lib.Hierarchy(A)

    def solve(st, h):
        with torch.cuda.stream(st):
            x = dev(b) * 0
            r = h.solve(dev(b), x, tol=1e-10, maxit=100)
            st.synchronize()
            return host(x), r.iters

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    handles = [on(st) for st in streams]
    use = [h.grid_use() for h in handles]
    first = use.count(2)
    assert use == [2] * first + [0] * (16 - first) and 0 < first <= cus // 33
    want, iters = solve(streams[0], handles[0])
    for st, h in list(zip(streams, handles))[1:]:
        x, it = solve(st, h)
        assert it == iters and abs(x - want).max() <= 1e-10 * abs(want).max()
    more = [on(streams[0]) for _ in range(3)]            # a stream that has its place
    assert [h.grid_use() for h in more] == [2] * 3
    handles[0].close()
    assert on(streams[15]).grid_use() == 0               # still used by the three
    for h in more:
        h.close()
    idle = [on(st) for st in streams[1:]]                # neither cycles nor solves: no place taken
    late = on(streams[15])
    assert late.grid_use() == 2 and handles[15].grid_use() == 0
    assert len(idle) == 15
