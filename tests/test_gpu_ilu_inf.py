"""An infinite entry of the factor whose value a block reads from memory: the row's result is infinite, as
plain substitution gives it, and not a NaN."""
import numpy as np
import pytest
import scipy.sparse as sp

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1106_3678_amd import binding  # noqa: E402


def test_infinite_entry_of_another_block():
    N, row = 1000, 900   # blocks of 640 rows; 4 entries a row on one side: 2 are packed
    A = sp.lil_matrix(sp.diags([np.full(N - k, -0.1) for k in (4, 3, 2, 1)] + [np.full(N, 2.0)], [-4, -3, -2, -1, 0]))
    A[1:5, 0] = 0.0
    A[row, row - 4:row] = 0.0
    A[0, 0] = 1e-10
    A[row, 0] = 1e308    # the row's only entry: l = a / u overflows
    A = sp.csr_matrix(A)
    A.eliminate_zeros()
    v = np.ones(N)
    with np.errstate(over="ignore"):
        L = A.toarray() / A.diagonal()
    y = np.zeros(N)
    for i in range(N):
        y[i] = v[i]
        for j in np.nonzero(L[i, :i])[0]:
            y[i] -= L[i, j] * y[j]
    ref = y / A.diagonal()
    assert np.isinf(ref[row]) and not np.any(np.isnan(ref))
    s = binding.Solver(binding.to_device(A), 2, tol=1e-10, maxit=100, precond=binding.MLB_PRECOND_ILU0)
    x, out = torch.from_numpy(v).cuda(), torch.zeros(N, dtype=torch.float64, device="cuda")
    s.matvec(x, out, binding.MLB_OP_MINV)
    got = out.cpu().numpy()
    s.close()
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.array_equal(np.sign(got), np.sign(ref))
    assert np.allclose(got[~np.isinf(ref)], ref[~np.isinf(ref)], rtol=1e-13)
