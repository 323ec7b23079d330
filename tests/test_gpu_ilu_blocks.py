"""The triangular solves of ILU(0) by blocks of rows: patterns at the edges of their paths.

A workgroup takes a block of consecutive rows by level, in chunks of at most 64 rows of one level.
Values of its own block come from a ring in LDS, those far behind and those of other blocks from
memory; a row's first entries are packed, the others read from the factor.  One application of
M^{-1} and M^{-H} element by element against the oracle's, with the bar of the other application
tests (1e-12 of the largest entry; both sides substitute the same factor)."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads
from tests.gpu_util import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from tests.test_gpu_ilu import _apply_both, _random_rows  # noqa: E402


def _csr(rows, cols, N, seed):
    """Off-diagonal entries at (rows, cols) and at their transposes, a dominant diagonal."""
    g = np.random.default_rng(seed)
    r = np.concatenate([rows, cols, np.arange(N)])
    c = np.concatenate([cols, rows, np.arange(N)])
    v = np.concatenate([g.standard_normal(2 * len(rows)), np.zeros(N)])
    A = sp.csr_matrix((v, (r, c)), shape=(N, N))
    A = (A + sp.diags(np.asarray(abs(A).sum(axis=1)).ravel() + 1.0)).tocsr()
    A.sort_indices()
    return workloads.Problem("pattern", A, np.ones(N), np.ones((N, 1)), np.zeros(N), 1, 1e-10, 100)


def chain(N):
    """Tridiagonal: every level, and every chunk, is one row."""
    i = np.arange(1, N)
    return _csr(i, i - 1, N, 1)


def far_in_block(N=160000, block=8000):
    """Blocks of 8,000 rows whose last 1,000 read rows 7,000 positions behind: past the ring's reach."""
    i = np.arange(N)
    i = i[i % block >= 7000]
    return _csr(i, i - 7000, N, 2)


def arrow(N):
    """Every row reads row 0, and the last 70 rows 50 rows each: entries past the 31st of a row."""
    i = np.arange(1, N)
    g = np.random.default_rng(3)
    r = np.repeat(np.arange(N - 70, N), 50)
    c = np.concatenate([g.choice(np.arange(1, N - 70), 50, replace=False) for _ in range(70)])
    return _csr(np.concatenate([i, r]), np.concatenate([np.zeros(N - 1, dtype=int), c]), N, 3)


CASES = {
    "chain": lambda: chain(3000),
    "far_in_block": far_in_block,
    "arrow": lambda: arrow(2500),
    "diagonal": lambda: _csr(np.array([], dtype=int), np.array([], dtype=int), 3000, 4),
    "one_over_a_block": lambda: chain(641),
    "grid_ragged": lambda: workloads.config2(n=1, m=33),
    "dense_rows": lambda: _random_rows(700, 60, 5),
    "blocks_dense_rows": lambda: _random_rows(900, 40, 6, block=True),
}


@pytest.mark.parametrize("case", list(CASES))
def test_apply(case):
    y, yh, y2, yo, yho = _apply_both(CASES[case]())
    for a, ref in ((y, yo), (yh, yho)):
        assert np.all(np.isfinite(a))
        assert np.max(np.abs(a - ref)) <= 1e-12 * np.max(np.abs(ref)), case
    assert np.array_equal(y, y2), case
