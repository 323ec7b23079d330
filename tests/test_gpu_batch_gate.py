"""A batch whose groups leave at their gate (MLB_GRID_ENTRY_TICKS=0: a group that is not complete at once
leaves) is solved all the same: the one-slice systems in their launch, the others by launches in the end."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402


@pytest.mark.parametrize("sides", [(90,), (90, 16, 40, 16, 75)])
def test_groups_that_leave(sides, monkeypatch):
    monkeypatch.setenv("MLB_GRID_ENTRY_TICKS", "0")
    g = np.random.default_rng(4)
    items = []
    for m in sides:
        A = workloads.convdiff_2d(m, pe=5.0)
        b, q = A @ g.standard_normal(m * m), np.asfortranarray(g.standard_normal((m * m, 2)))
        items.append((A, b, binding.Solver(binding.to_device(A), 2, tol=1e-10, maxit=4000),
                      torch.from_numpy(b).cuda(), torch.zeros(m * m, dtype=torch.float64, device="cuda"),
                      binding.column_major(q)))
    res = binding.solve_batch([i[2] for i in items], [i[3] for i in items], [i[4] for i in items],
                              [i[5] for i in items])
    torch.cuda.synchronize()
    for r, (A, b, s, _, x, _) in zip(res, items):
        true = np.linalg.norm(b - A @ x.cpu().numpy()) / np.linalg.norm(b)
        # the stop is on the recursive residual; the true one follows it closely at these sizes
        assert r.flag == 0 and r.err_recursive < 1e-10 and abs(r.err_true - true) < 1e-12 and true < 1e-8
        s.close()
