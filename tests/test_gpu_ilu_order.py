"""ILU(0)'s triangular solves by level, for patterns that blocks of rows do not suit, and blocks of rows on
the patterns at the edge of the rule.  One application of M^{-1} and M^{-H} element by element against the
oracle's, with the bar of the other application tests (1e-12 of the largest entry; both sides substitute the
same factor), and the time of such patterns against one that suits blocks."""
import time

import numpy as np
import pytest
import scipy.sparse as sp

import workloads
from tests.gpu_util import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_1106_3678_amd import binding  # noqa: E402
from tests.test_gpu_ilu import _apply_both  # noqa: E402


def matrix(rows, cols, N, seed, cplx=False, blocks=False):
    """Off-diagonal entries at (rows, cols) and at their transposes, a dominant diagonal."""
    g = np.random.default_rng(seed)
    A = sp.csr_matrix((np.ones(len(rows)), (rows, cols)), shape=(N, N))
    A = sp.csr_matrix(A + A.T)
    A.data = g.standard_normal(A.nnz) + (1j * g.standard_normal(A.nnz) if cplx else 0)
    A = sp.csr_matrix(A + sp.diags(np.asarray(abs(A).sum(axis=1)).ravel() + 1.0))
    A.sort_indices()
    if blocks:
        A = sp.kron(A, np.eye(3) + 0.1 * g.standard_normal((3, 3)), format="bsr")
        A.sort_indices()
    return A


def grid(m, order=None):
    """Neighbours on an m^3 grid, in natural order, red-black or random."""
    i = np.arange(m ** 3)
    x, y, z = i % m, i // m % m, i // m // m
    r = np.concatenate([i[x > 0], i[y > 0], i[z > 0]])
    c = np.concatenate([i[x > 0] - 1, i[y > 0] - m, i[z > 0] - m * m])
    p = i
    if order == "red_black":
        p = np.argsort(np.argsort((x + y + z) % 2, kind="stable"), kind="stable")
    elif order == "random":
        p = np.random.default_rng(m).permutation(m ** 3)
    return np.maximum(p[r], p[c]), np.minimum(p[r], p[c])


def band(N, half):
    i = np.repeat(np.arange(N), half)
    j = i - np.tile(np.arange(1, half + 1), N)
    return i[j >= 0], j[j >= 0]


def scattered(N, k):
    g = np.random.default_rng(k)
    r = np.repeat(np.arange(1, N), k)
    return r, (g.random(r.size) * r).astype(int)


def chain_and(N, r, c):
    i = np.arange(1, N)
    return np.concatenate([i, r]), np.concatenate([i - 1, c])


def some_far(N=160000):
    """A chain, and one row in 20 reads the row 7,000 before it: in its block, beyond the ring."""
    i = np.arange(7000, N, 20)
    return chain_and(N, i, i - 7000)


def some_long(N=3000):
    """A chain with a few rows of 40 entries: past the 31st, and past the packed ones."""
    r = np.repeat(np.arange(1000, N, 500), 40)
    return chain_and(N, r, r - 2 - np.tile(np.arange(40), r.size // 40) * 20)


PATTERNS = {
    "red_black": (4096, lambda: grid(16, "red_black")),
    "random_order": (4096, lambda: grid(16, "random")),
    "natural": (4096, lambda: grid(16)),
    "scattered": (3000, lambda: scattered(3000, 6)),
    "two_diagonals": (5000, lambda: (np.arange(2000, 5000), np.arange(3000))),
    "band_40": (1500, lambda: band(1500, 40)),
    "some_long": (3000, some_long),
    "one_row": (1, lambda: (np.array([], dtype=int), np.array([], dtype=int))),
}


def check(A, N):
    N = A.shape[0]
    y, yh, y2, yo, yho = _apply_both(workloads.Problem("pattern", A, np.ones(N), np.ones((N, 1)), np.zeros(N), 1,
                                                       1e-10, 100))
    for a, ref in ((y, yo), (yh, yho)):
        assert np.all(np.isfinite(a))
        assert np.max(np.abs(a - ref)) <= 1e-12 * np.max(np.abs(ref))
    assert np.array_equal(y, y2)


@pytest.mark.parametrize("kind", ["real", "complex", "blocks"])
@pytest.mark.parametrize("name", list(PATTERNS))
def test_apply(name, kind):
    N, make = PATTERNS[name]
    check(matrix(*make(), N, 11, cplx=kind == "complex", blocks=kind == "blocks"), N)


def test_apply_beyond_the_ring():
    check(matrix(*some_far(), 160000, 12), 160000)


def test_apply_one_way_long_columns():
    """A long column: the factor goes by blocks, its transpose, with a long row, too or by level."""
    N = 4000
    i = np.arange(1, N)
    A = sp.csr_matrix((np.full(N - 1, 0.5), (i, i - 1)), shape=(N, N)) + sp.diags(np.full(N, 4.0))
    A = sp.lil_matrix(A)
    A[2000:, 5] = 0.25
    check(sp.csr_matrix(A), N)


def apply_us(A):
    dA = binding.to_device(A)
    v = torch.randn(A.shape[0], dtype=torch.float64, device="cuda")
    y = torch.empty_like(v)
    s = binding.Solver(dA, 1, tol=1e-10, maxit=10, precond=binding.MLB_PRECOND_ILU0)
    best = 1e9
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        s.matvec(v, y, binding.MLB_OP_MINV)
        best = min(best, time.perf_counter() - t)
    s.close()
    return best * 1e6


def test_red_black_is_not_slower_than_natural_order():
    """Two wide levels: by level the red-black grid takes half the natural order's time (150 us against 320);
    by blocks of rows it took 0.9 of it."""
    natural = apply_us(matrix(*grid(64), 64 ** 3, 1))
    red_black = apply_us(matrix(*grid(64, "red_black"), 64 ** 3, 1))
    print(f"natural {natural:.0f} us, red-black {red_black:.0f}", flush=True)
    assert red_black < 0.7 * natural
