"""A system of a batch gives bitwise what it gives alone, whatever variant of the kernel its neighbours' shadow
vectors or sizes ask for: rows of more than one batch of entries, 4 shadow vectors beside 8, 9 and 17, one slice
beside many."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402
from tests.test_gpu_grid import random_problem  # noqa: E402


def prepare(p, tf=False):
    dA, b, Q = binding.to_device(p.A), torch.from_numpy(p.b).cuda(), binding.column_major(p.Q)
    return binding.Solver(dA, p.n, tol=p.tol, maxit=p.maxit, transpose_free=tf), b, Q


def run(items):
    xs = [torch.zeros_like(b) for _, b, _ in items]
    rs = binding.solve_batch([s for s, _, _ in items], [b for _, b, _ in items], xs, [q for _, _, q in items])
    torch.cuda.synchronize()
    return [(r.flag, r.iter, r.err_recursive, r.err_true) for r in rs], [x.clone() for x in xs]


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("tf", [False, True])
@pytest.mark.parametrize("per_row", [5, 13, 16, 21])
@pytest.mark.parametrize("other_n", [8, 9, 17])
def test_beside_more_shadow_vectors(per_row, other_n, tf, cplx):
    me = prepare(random_problem(1111, per_row, 4, 900 + per_row, cplx=cplx), tf)
    other = prepare(random_problem(700, 6, other_n, 950 + other_n, cplx=cplx), tf)
    alone, xa = run([me])
    mixed, xm = run([other, me])
    for s, _, _ in (me, other):
        s.close()
    assert alone[0][0] == 0 and mixed[1] == alone[0]
    assert torch.equal(xm[1], xa[0])


def test_beside_a_system_of_many_rows():
    """140,625 rows take more than one row a thread, so the small system runs from memory, too."""
    me = prepare(random_problem(1111, 5, 4, 905))
    A = workloads.convdiff_2d(375, pe=40.0)
    g = np.random.default_rng(1)
    big = workloads.Problem("big", A, A @ g.standard_normal(A.shape[0]), np.asfortranarray(
        g.standard_normal((A.shape[0], 2))), None, 2, 1e-4, 20000)
    other = prepare(big)
    alone, xa = run([me])
    mixed, xm = run([other, me])
    for s, _, _ in (me, other):
        s.close()
    assert alone[0][0] == 0 and mixed[1] == alone[0] and torch.equal(xm[1], xa[0])
