"""A solve in which any workgroup lost a wait is reported as an error, and never returns an x some of whose
rows were not stored.  MLB_GRID_MAX_TRIES bounds the tries of a wait, so that some waits of some solves are lost.
(A loss long after the last sums are out, when the first workgroup already has its result, cannot be forced
this way; the host sees it by the word that every workgroup that lost a wait writes.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402


@pytest.mark.parametrize("m", [32, 90])   # 2 and 16 slices
def test_lost_wait_is_never_a_result(m, monkeypatch):
    A = workloads.convdiff_2d(m, pe=5.0)
    g = np.random.default_rng(3)
    dA = binding.to_device(A)
    b = torch.from_numpy(g.standard_normal(m * m)).cuda()
    Q = binding.column_major(g.standard_normal((m * m, 2)))
    x = torch.zeros_like(b)

    def solver():   # block Jacobi: the launch leaves no residual, so the last sums are the recurrence's
        return binding.Solver(dA, 2, tol=1e-12, maxit=2, precond=binding.MLB_PRECOND_JACOBI)

    s = solver()
    assert s.solve(b, x, Q).flag == 1
    s.close()
    ref, done, lost = x.clone(), 0, 0
    for tries in range(1, 60):
        monkeypatch.setenv("MLB_GRID_MAX_TRIES", str(tries))
        s = solver()
        for _ in range(40):
            x.zero_()
            try:
                flag = s.solve(b, x, Q).flag
            except binding.MlbError as e:
                assert e.code == binding.MLB_EHIP
                lost += 1
                continue
            done += 1
            assert flag == 1 and torch.equal(x, ref), tries
        s.close()
    print(f"{m}: {done} solved, {lost} lost", flush=True)
    assert lost > 0
