"""Solves whose matrix has rows too long for one lane are iterated by launches.  The route is shown by the
whole-solve kernel's own test hook: with MLB_GRID_MAX_TRIES=1 every wait of it that is not over at its first
look is lost, so a solve of several slices that goes through it ends in MLB_EHIP.  A batch, which has no other
kernel, always goes through it.  Results against scipy's direct solver (diagonally dominant systems: the bar
is the solve's tolerance times a small factor)."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg as spla

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1106_3678_amd import binding  # noqa: E402

N = 2046   # four slices of 512; divisible by 3 for the blocks


def with_entries(rows, cols, cplx=False, blocks=False):
    g = np.random.default_rng(len(rows))
    m = N // 3 if blocks else N
    off = rows != cols
    rows, cols = rows[off], cols[off]
    A = sp.csr_matrix((g.standard_normal(len(rows)) + 0.1, (rows, cols)), shape=(m, m))
    A.sum_duplicates()
    A = sp.csr_matrix(A + sp.diags(2.0 + np.asarray(abs(A).sum(axis=1)).ravel()))
    if cplx:
        A = sp.csr_matrix(A * (1 + 0.5j))
    return sp.kron(A, np.eye(3) + 0.1, format="bsr") if blocks else A


def even(per_row, **kw):
    """per_row entries in every row, cyclically behind the diagonal."""
    m = N // 3 if kw.get("blocks") else N
    i = np.repeat(np.arange(m), per_row)
    return with_entries(i, (i + np.tile(np.arange(per_row), m)) % m, **kw)


def one_row(length, transpose=False, blocks=False):
    """Three entries a row, one row (or column) of `length`."""
    m = N // 3 if blocks else N
    i = np.repeat(np.arange(m), 3)
    j = (i + np.tile([0, 1, m - 1], m)) % m
    keep = i != 700 % m
    if transpose:
        keep = j != 700 % m
    k = np.arange(length)
    r, c = np.concatenate([i[keep], np.full(length, 700 % m)]), np.concatenate([j[keep], (700 % m + k) % m])
    if transpose:
        r, c = np.concatenate([i[keep], (700 % m + k) % m]), np.concatenate([j[keep], np.full(length, 700 % m)])
    return with_entries(r, c, blocks=blocks)


CASES = {   # matrix, n, solved by launches
    "47_a_row": (lambda: even(47), 4, False),
    "48_a_row": (lambda: even(48), 4, True),
    "8_a_row": (lambda: even(8), 4, False),
    "complex_16_shadow_vectors": (lambda: even(5, cplx=True), 16, False),
    "complex_17_shadow_vectors": (lambda: even(5, cplx=True), 17, True),
    "complex_31": (lambda: even(31, cplx=True), 4, False),
    "complex_32": (lambda: even(32, cplx=True), 4, True),
    "blocks_27": (lambda: even(27, blocks=True), 4, False),
    "blocks_28": (lambda: even(28, blocks=True), 4, True),
    "row_96": (lambda: one_row(96), 4, False),
    "row_97": (lambda: one_row(97), 4, True),
    "block_row_48": (lambda: one_row(48, blocks=True), 4, False),
    "block_row_49": (lambda: one_row(49, blocks=True), 4, True),
    "column_1365": (lambda: one_row(1365, True), 4, False),
    "column_1366": (lambda: one_row(1366, True), 4, True),
    "column_1366_n3": (lambda: one_row(1366, True), 3, False),
}


def solve(A, n, batch=False):
    g = np.random.default_rng(7)
    cplx = np.iscomplexobj(A.data)
    rnd = lambda *s: g.standard_normal(s) + (1j * g.standard_normal(s) if cplx else 0)
    b, Qh = rnd(N), rnd(N, n)
    dA = binding.to_device(A)
    bd, Q = torch.from_numpy(b).cuda(), binding.column_major(Qh)
    x = torch.zeros_like(bd)
    s = binding.Solver(dA, n, tol=1e-10, maxit=500)
    try:
        r = binding.solve_batch([s], [bd], [x], [Q])[0] if batch else s.solve(bd, x, Q)
    finally:
        s.close()
    torch.cuda.synchronize()
    return r, x.cpu().numpy(), b


@pytest.mark.parametrize("case", list(CASES))
def test_route_and_result(case, monkeypatch):
    make, n, launches = CASES[case]
    A = make()
    r, x, b = solve(A, n)
    ref = spla.spsolve(sp.csc_matrix(A), b)
    assert r.flag == 0 and np.linalg.norm(x - ref) <= 1e-8 * np.linalg.norm(ref)
    monkeypatch.setenv("MLB_GRID_MAX_TRIES", "1")
    if launches:
        assert solve(A, n)[0].flag == 0
        if A.format == "csr":
            with pytest.raises(binding.MlbError):
                solve(A, n, batch=True)
    else:
        with pytest.raises(binding.MlbError) as e:
            solve(A, n)
        assert e.value.code == binding.MLB_EHIP
