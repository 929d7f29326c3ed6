"""Row-by-row products and transposes of the device setup (product_kernels.hip)
where a row outgrows what it is given: the first kernel's table, the second's
(then the terms are sorted), the terms a row may have, the entries a row of the
transpose may have, and the rows a wave stages.  Every level equals
the oracle's bit for bit, as in the other tests of the device setup."""
import numpy as np
import pytest
from scipy import sparse

from paper_1512_04629_amd import inputs as I

from .test_gpu_setup_device import lib, oracle, same_hierarchy  # noqa: F401

pytestmark = pytest.mark.gpu


def csr(i, j, v, n):
    """The Laplacian of weighted edges, plus a hundredth on the diagonal."""
    m = sparse.coo_matrix((np.r_[-v, -v], (np.r_[i, j], np.r_[j, i])), shape=(n, n)).tocsr()
    m = (m + sparse.diags_array(0.01 - np.asarray(m.sum(axis=1)).ravel())).tocsr()
    m.sort_indices()
    return I.CSR(n, m.indptr.astype(np.int32), m.indices.astype(np.int32), m.data.astype(np.float64))


def arrow(n, links):
    """A chain of n points, the first `links` of them weakly coupled to a hub that
    depends on a partner: the hub's rows of A P and of P^T A P have about half as
    many columns as it has links, its interpolation one."""
    c, k = np.arange(n - 1), np.arange(links)
    w = 1.0 + 0.25 * I.uniform01(3, n - 1)
    i = np.r_[c, k, n]
    j = np.r_[c + 1, np.full(links, n), n + 1]
    return csr(i, j, np.r_[w, np.full(links, 2.0**-10), [1000.0]], n + 2)


def star(leaves):
    """A hub every leaf depends on: one column of P, one row of R."""
    k = np.arange(1, leaves + 1)
    return csr(np.zeros(leaves, int), k, np.ones(leaves), leaves + 1)


def dense(n):
    """Every point coupled to every other."""
    i, j = np.triu_indices(n, 1)
    return csr(i, j, 0.5 + I.uniform01(5, len(i)), n)


CASES = {
    "one_row": lambda: csr(np.array([0]), np.array([1]), np.array([1.0]), 2),
    "first_table_full": lambda: arrow(400, 90),
    "second_table": lambda: arrow(2000, 900),
    "more_columns_than_a_table": lambda: arrow(3000, 1300),
    "more_terms_than_a_row": lambda: arrow(8000, 8000),
    "dense_levels_of_20_million_entries": lambda: arrow(24000, 24000),
    "row_of_the_transpose_2047": lambda: star(2047),
    "row_of_the_transpose_2048": lambda: star(2048),
    "row_of_the_transpose_40000": lambda: star(40000),
    "long_rows": lambda: dense(300),
}


@pytest.mark.parametrize("name,coarsening", [(k, "pmis") for k in sorted(CASES)] +
                         [(k, "rs") for k in ("long_rows", "row_of_the_transpose_2048", "second_table")])
def test_long_rows_equal_oracle(lib, name, coarsening):  # noqa: F811
    A = CASES[name]()
    kw = dict(max_coarse=1) if A.n < 100 else {}
    g = lib.Hierarchy(A, setup="device", coarsening=coarsening, seed=2, **kw)
    o = oracle(A, coarsening="pmis", seed=2, **kw) if coarsening == "pmis" else oracle(A, **kw)
    same_hierarchy(g, o, o.cf)
