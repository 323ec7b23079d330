"""Which served requests are solved in one launch and which by launches, shown by the whole-solve kernel's
own test hook: with MLB_GRID_MAX_TRIES=1 every wait of it that is not over at its first look is lost, so a
request that goes through it (with more than one slice of 512 rows) ends in MLB_EHIP, and one that is
iterated by launches is solved."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402


def serve(m, precision=0):
    p = workloads.serving_problem(workloads.Request(0, 0.0, 2, m, 5.0, 4, 500 + m), tol=1e-6)
    dA, b, Q = binding.to_device(p.A), torch.from_numpy(p.b).cuda(), binding.column_major(p.Q)
    x = torch.zeros_like(b)
    torch.cuda.synchronize()
    server = binding.Server(budget_bytes=4 << 30, max_inflight=1)
    try:
        return server.wait(server.submit(dA, b, x, Q, p.n, tol=p.tol, maxit=p.maxit, precision=precision))[0]
    finally:
        server.close()


@pytest.mark.parametrize("precision", [binding.MLB_PREC_FP64, binding.MLB_PREC_FP32_IR])
def test_large_requests_go_by_launches(precision, monkeypatch):
    """180,625 rows, beyond the line at 180,000: a group that would hold the card alone."""
    monkeypatch.setenv("MLB_GRID_MAX_TRIES", "1")
    assert serve(425, precision).flag == 0


@pytest.mark.parametrize("m", [200, 424])
def test_small_requests_go_in_one_launch(m, monkeypatch):
    """40,000 rows, beyond the batchers' sizes, and 179,776, before the line."""
    monkeypatch.setenv("MLB_GRID_MAX_TRIES", "1")
    with pytest.raises(binding.MlbError) as e:
        serve(m)
    assert e.value.code == binding.MLB_EHIP
