"""Two ILU(0) solvers alive at once whose blocks need different amounts of LDS (one and four packed entries a
row): each gives the same before the other is there, beside it, and after it is gone."""
import numpy as np
import pytest
import scipy.sparse as sp
import scipy.sparse.linalg  # noqa: F401

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_1106_3678_amd import binding  # noqa: E402


def band(N, half, cplx):
    k = np.arange(-half, half + 1)
    A = sp.diags([np.full(N - abs(j), -1.0 / (1 + abs(j)) if j else 4.0) for j in k], k).tocsr()
    return A * (1 + 0.5j) if cplx else A


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("first,second", [(4, 1), (1, 4)])
def test_two_factors(first, second, cplx):
    N = 5000
    g = np.random.default_rng(0)
    v = torch.from_numpy(g.standard_normal(N) + (1j * g.standard_normal(N) if cplx else 0)).cuda()

    def make(half):
        return binding.Solver(binding.to_device(band(N, half, cplx)), 2, tol=1e-10, maxit=100,
                              precond=binding.MLB_PRECOND_ILU0)

    def apply(s, op):
        y = torch.zeros_like(v)
        s.matvec(v, y, op)
        return y

    ops = (binding.MLB_OP_MINV, binding.MLB_OP_MINVH)
    a = make(first)
    alone = [apply(a, op) for op in ops]
    b = make(second)
    other = [apply(b, op) for op in ops]
    assert all(torch.equal(apply(a, op), y) for op, y in zip(ops, alone))
    assert all(torch.equal(apply(b, op), y) for op, y in zip(ops, other))
    b.close()
    assert all(torch.equal(apply(a, op), y) for op, y in zip(ops, alone))
    # a band is its own LU pattern, so M^{-1} is A^{-1}
    ref = sp.linalg.spsolve(sp.csc_matrix(band(N, first, cplx)), v.cpu().numpy())
    assert np.linalg.norm(alone[0].cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)
    a.close()
