"""An initial guess that holds the bit pattern by which a whole solve marks words as pending: a NaN like any
other, so the solve ends with a breakdown (-1) at once and leaves x as it was."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402

PATTERN = 0x7FF00000000000A5


@pytest.mark.parametrize("m", [8, 40, 400])   # one slice, four, and 256 of more than a row a thread
@pytest.mark.parametrize("kind", ["real", "complex", "batch"])
def test_pending_pattern_in_x0(m, kind):
    A = workloads.convdiff_2d(m, pe=5.0)
    cplx = kind == "complex"
    if cplx:
        A = A * (1 + 0.25j)
    g = np.random.default_rng(m)
    N = A.shape[0]
    dt = torch.complex128 if cplx else torch.float64
    b = torch.from_numpy(g.standard_normal(N)).to(dt).cuda()
    Q = binding.column_major(g.standard_normal((N, 4)) + (0j if cplx else 0))
    x = torch.zeros(N, dtype=dt, device="cuda")
    words = (torch.view_as_real(x) if cplx else x).reshape(-1).view(torch.int64)
    words[words.numel() // 2] = PATTERN
    before = words.clone()
    s = binding.Solver(binding.to_device(A), 4, tol=1e-10, maxit=100)
    try:
        r = binding.solve_batch([s], [b], [x], [Q])[0] if kind == "batch" else s.solve(b, x, Q)
    finally:
        s.close()
    torch.cuda.synchronize()
    assert r.flag == -1 and r.iter == 0 and not np.isfinite(r.err_true)
    assert torch.equal(words, before)
