"""Served requests on both sides of the size from which a server worker iterates by launches (130,560
rows): each result is the same alone and beside others, and solves its system."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402

MESH = [361, 362]   # 130,321 and 131,044 rows: 255 and 256 slices of 512


def upload(m):
    p = workloads.serving_problem(workloads.Request(0, 0.0, 2, m, 5.0, 4, 500 + m), maxit=8000)
    return p, binding.to_device(p.A), torch.from_numpy(p.b).cuda(), binding.column_major(p.Q)


def serve(reqs, inflight):
    server = binding.Server(budget_bytes=8 << 30, max_inflight=inflight)
    xs = [torch.zeros_like(b) for _, _, b, _ in reqs]
    torch.cuda.synchronize()
    ts = [server.submit(dA, b, x, Q, p.n, tol=1e-8, maxit=p.maxit) for (p, dA, b, Q), x in zip(reqs, xs)]
    out = [server.wait(t)[0] for t in ts]
    server.close()
    return out, xs


@pytest.mark.parametrize("m", MESH)
def test_large_request_alone_and_in_a_mix(m):
    me = upload(m)
    others = [upload(k) for k in MESH]
    (alone,), (xa,) = serve([me], 1)
    mixed, xm = serve([me] + others, 3)
    assert alone.flag == 0 and mixed[0].flag == 0
    assert mixed[0].iter == alone.iter and torch.equal(xm[0], xa)
    # the recursive residual stops below 1e-8; the true one follows it to far less than that
    assert alone.err_true <= 2e-8
