"""A served ILU(0) request whose packed rows would exceed the budget, and that fits it with solves by level, is
admitted and solved; one that does not fit then is refused.  7-point 20^3: the larger form takes 40% more."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402

ILU = binding.MLB_PRECOND_ILU0


def by_level_bytes(p, n):
    """What a solver with solves by level takes: the workspace without packed rows (per row and solve: three
    indices, w entries with theirs, w = 3 on a 7-point grid), diagonals and the second vector in solve order."""
    opt = binding.mlb_options(n, p.tol, p.maxit, 0.0, 0, 0.0, 0, 0, None, ILU, 0, 0, 0)
    full = binding.mlbicgstab_workspace_size(binding.to_device(p.A).descriptor(), opt)
    return full - p.N * (4 * (12 + 3 * 12) + 2 * 8 + 8), full


@pytest.mark.parametrize("sequence", [False, True])
def test_budget_between(sequence):
    p = workloads.config2(n=4, m=20)
    level, full = by_level_bytes(p, 4)
    assert level < 0.8 * full
    dA, b, Q = binding.to_device(p.A), torch.from_numpy(p.b).cuda(), binding.column_major(p.Q)

    def serve(budget):
        x = torch.zeros_like(b)
        torch.cuda.synchronize()
        server = binding.Server(budget_bytes=budget, max_inflight=1)
        try:
            if sequence:
                t = server.submit_sequence(7, dA, b, x, Q, 4, 4, 4, 0, tol=p.tol, maxit=p.maxit, precond=ILU)
            else:
                t = server.submit(dA, b, x, Q, 4, tol=p.tol, maxit=p.maxit, precond=ILU)
            res, tim = server.wait(t)
            if sequence:
                server.end_sequence(7)
        finally:
            server.close()
        return res, tim.footprint_bytes, x.cpu().numpy()

    usual, fp, x = serve(full)
    assert usual.flag == 0 and fp == full
    lean, fp_lean, x_lean = serve(level)
    assert lean.flag == 0 and fp_lean == level and abs(lean.iter - usual.iter) <= max(1, usual.iter // 20)
    assert np.linalg.norm(x - x_lean) <= 1e-7 * np.linalg.norm(x)
    with pytest.raises(binding.MlbError) as e:
        serve(level - 1)
    assert e.value.code == binding.MLB_ENOMEM
