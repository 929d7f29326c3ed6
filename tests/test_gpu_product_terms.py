"""Products through sorted terms whose coarse rows hold thousands of them: the terms
are listed entry by entry, 4, 16 or 64 lanes an entry (by their mean number), and
every level equals the oracle's bit for bit."""
import pytest

from paper_1512_04629_amd import inputs as I

from .test_gpu_product import arrow, dense
from .test_gpu_setup_device import lib, oracle, same_hierarchy  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = {
    "few_terms_an_entry": lambda: arrow(9000, 9000),          # 4 lanes, one row of most
    "graph_2000": lambda: I.random_graph_laplacian(2000),     # 16 and 64 lanes
    "graph_9001": lambda: I.random_graph_laplacian(9001),
    "dense_701": lambda: dense(701),                          # 64 lanes, rows past them
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_listed_terms_equal_oracle(lib, name):  # noqa: F811
    A = CASES[name]()
    g = lib.Hierarchy(A, setup="device", coarsening="pmis", seed=3)
    o = oracle(A, coarsening="pmis", seed=3)
    same_hierarchy(g, o, o.cf)
