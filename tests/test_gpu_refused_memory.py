"""Allocations that the caller's allocator refuses: the call says so
(AMG_ERR_OUT_OF_MEMORY), nothing it had taken stays with the allocator, and no
kernel gets an array that is not there."""
import ctypes as C

import numpy as np
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_parity import dev

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

OUT_OF_MEMORY = -3


@pytest.fixture(scope="module")
def lib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_04629_amd import amg
    return amg.load_library()


class Refusing:
    """Refuses the allocation number `at` (from 1) after arm(at); none without."""

    def __init__(self):
        from paper_1512_04629_amd import amg
        self.count, self.at, self.live = 0, 0, {}

        def alloc(nbytes, stream, user):
            self.count += 1
            if self.count == self.at:
                return None
            p = torch.cuda.caching_allocator_alloc(int(nbytes), stream=int(stream or 0))
            self.live[p] = nbytes
            return p

        def free(ptr, nbytes, stream, user):
            del self.live[ptr]
            torch.cuda.caching_allocator_delete(ptr)

        self.alloc_fn, self.free_fn = amg.ALLOC_FN(alloc), amg.FREE_FN(free)

    def arm(self, at):
        self.count, self.at = 0, at

    @property
    def refused(self):
        return 0 < self.at <= self.count


def stream():
    return C.c_void_p(torch.cuda.current_stream().cuda_stream)


def on_host(lib, A, mem):
    rp, ci = np.ascontiguousarray(A.row_ptr, np.int32), np.ascontiguousarray(A.col, np.int32)
    v, h = np.ascontiguousarray(A.val, np.float64), C.c_void_p()
    st = lib.amg_setup_from_csr(A.n, rp.ctypes.data, ci.ctypes.data, v.ctypes.data, None, stream(), mem.alloc_fn,
                                mem.free_fn, None, C.byref(h))
    return st, h


def on_device(lib, csr, mem):
    n, rp, ci, v = csr
    h = C.c_void_p()
    st = lib.amg_setup_device(n, ci.numel(), rp.data_ptr(), ci.data_ptr(), v.data_ptr(), None, 1, 1, stream(),
                              mem.alloc_fn, mem.free_fn, None, C.byref(h))
    return st, h


def device_csr(A):
    return (A.n, torch.from_numpy(np.ascontiguousarray(A.row_ptr, np.int32)).cuda(),
            torch.from_numpy(np.ascontiguousarray(A.col, np.int32)).cuda(), dev(A.val))


CASES = {
    # the fine operators large enough for the stored forms (SELL-64 copies, pair codes)
    "device_large": (on_device, lambda: device_csr(I.poisson3d(64))),
    "device_values": (on_device, lambda: device_csr(I.fv3d_lognormal(64))),
    # levels that one launch takes
    "host_small": (on_host, lambda: I.poisson2d(40)),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_a_setup_that_fails_gives_everything_back(lib, name):
    make, problem = CASES[name]
    A = problem()
    mem = Refusing()
    at = 1
    while True:
        mem.arm(at)
        st, h = make(lib, A, mem)
        if not mem.refused:
            break
        assert st == OUT_OF_MEMORY and not h.value, at
        assert not mem.live, (at, sorted(mem.live.values()))
        at += 1
    assert st == 0 and at > 30
    lib.amg_destroy(h)
    assert not mem.live


def solve(lib, h, A, b, precision=64):
    from paper_1512_04629_amd import amg
    p, info = amg.SolveParams(1, 1e-10, 100, 0, 3, 1, 0.5, 0.01, precision, 0), amg.SolveInfo()
    x = torch.zeros(A.n, dtype=torch.float64, device="cuda")
    st = lib.amg_solve(h, b.data_ptr(), x.data_ptr(), C.byref(p), C.byref(info), None)
    assert st == 0, lib.amg_last_error(h)
    return x.cpu().numpy()


@pytest.mark.parametrize("strong", [0, 1])
def test_a_sparsification_that_fails_can_be_repeated(lib, strong):
    A = I.poisson3d(20)
    b = dev(I.rhs(A.n, 3))

    def make(fp32):
        mem = Refusing()
        st, h = on_host(lib, A, mem)
        assert st == 0
        solve(lib, h, A, b, 32 if fp32 else 64)
        assert lib.amg_set_lumping(h, strong) == 0
        return mem, h

    for fp32 in (False, True):
        mem, h = make(fp32)
        assert lib.amg_sparsify(h, 0.1, 2) == 0
        want = solve(lib, h, A, b), solve(lib, h, A, b, 32)
        lib.amg_destroy(h)
        at = 1
        while True:
            mem, h = make(fp32)
            mem.arm(at)
            st = lib.amg_sparsify(h, 0.1, 2)
            refused = mem.refused
            assert st == (OUT_OF_MEMORY if refused else 0), at
            mem.arm(0)
            if refused:
                for precision in (64, 32):        # the hierarchy as it was
                    solve(lib, h, A, b, precision)
                assert lib.amg_sparsify(h, 0.1, 2) == 0
                assert np.array_equal(solve(lib, h, A, b), want[0])
                assert np.array_equal(solve(lib, h, A, b, 32), want[1])
            lib.amg_destroy(h)
            assert not mem.live
            if not refused:
                break
            at += 1
        assert at > 6


@pytest.mark.parametrize("name", ["device_large", "device_values"])
def test_a_switch_of_forms_that_fails(lib, name):
    """Every operator is served by one form or another afterwards, and the switch can
    be repeated."""
    make, problem = CASES[name]
    csr = problem()
    A = I.poisson3d(64) if name == "device_large" else I.fv3d_lognormal(64)
    b = dev(I.rhs(A.n, 3))
    mem = Refusing()
    st, h = make(lib, csr, mem)
    assert st == 0
    want = {}
    for on in (1, 0, 1):
        assert lib.amg_set_compact_indices(h, on) == 0
        want[on] = solve(lib, h, A, b), solve(lib, h, A, b, 32)
    at, tried = 1, 0
    while True:
        refused = 0
        for on in (0, 1):
            mem.arm(at)
            st = lib.amg_set_compact_indices(h, on)
            assert st == (OUT_OF_MEMORY if mem.refused else 0), (at, on)
            if mem.refused:
                refused += 1
                mem.arm(0)
                assert np.allclose(solve(lib, h, A, b), want[1][0], rtol=0, atol=1e-8 * abs(want[1][0]).max())
                assert np.allclose(solve(lib, h, A, b, 32), want[1][0], rtol=0, atol=1e-7 * abs(want[1][0]).max())
                assert lib.amg_set_compact_indices(h, on) == 0
            mem.arm(0)
            assert np.array_equal(solve(lib, h, A, b), want[on][0])
            assert np.array_equal(solve(lib, h, A, b, 32), want[on][1])
        tried += 1
        at += 1
        if not refused:
            break
    lib.amg_destroy(h)
    assert not mem.live and tried > 2
