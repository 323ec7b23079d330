"""Solves on a stream of the caller's own: a group of more than half the card's CUs is iterated by launches
there, and in one launch on the default stream; smaller groups and batches always in one launch.  The route
is shown by the whole-solve kernel's own test hook: with MLB_GRID_MAX_TRIES=1 every wait of it that is not over
at its first look is lost, so a solve of several slices that goes through it ends in MLB_EHIP."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402


def solve(m, stream=None, batch=False, precision=0, noalloc=False):
    p = workloads.serving_problem(workloads.Request(0, 0.0, 2, m, 5.0, 2, 700 + m), tol=1e-4)
    dA, b, Q = binding.to_device(p.A), torch.from_numpy(p.b).cuda(), binding.column_major(p.Q)
    x = torch.zeros_like(b)
    torch.cuda.synchronize()
    s = binding.Solver(dA, p.n, tol=p.tol, maxit=p.maxit, stream=stream, precision=precision)
    try:
        r = binding.solve_batch([s], [b], [x], [Q])[0] if batch else s.solve(b, x, Q)
    finally:
        s.close()
    torch.cuda.synchronize()
    assert r.flag == 0 and np.linalg.norm(p.b - p.A @ x.cpu().numpy()) <= 2e-4 * np.linalg.norm(p.b)
    return x


# 65,536 rows are 128 slices of 512, 66,049 are 130 of at most 512
@pytest.mark.parametrize("m,own,kw,launches", [
    (256, True, {}, False), (257, True, {}, True), (257, False, {}, False), (257, True, {"batch": True}, False),
    (257, True, {"precision": 1}, True), (362, True, {"precision": 1}, True), (362, False, {"precision": 1}, False)])
def test_route(m, own, kw, launches, monkeypatch):
    monkeypatch.setenv("MLB_GRID_MAX_TRIES", "1")
    stream = torch.cuda.Stream() if own else None
    if launches:
        solve(m, stream, **kw)
    else:
        with pytest.raises(binding.MlbError) as e:
            solve(m, stream, **kw)
        assert e.value.code == binding.MLB_EHIP


def test_same_on_every_own_stream():
    a, b = solve(300, torch.cuda.Stream()), solve(300, torch.cuda.Stream())
    assert torch.equal(a, b)
