"""The sums of the fp32 iteration beyond a thread's rows are added in fp64.  A diagonal system of 1s and 2s whose
first step, half of it taken, leaves exactly the rows of the 2s: one of 2^-10 and seven of 2^-22 in each of 256
slices, each in a wave of its own.  In fp32 the seven squares, 2^-24 of the first, would be lost one by one, and
the norm come out 2.1e-7 too small, below an inner tolerance set 1.0e-7 below its true value: the inner solve would
stop on that half step and leave the refinement another step to do.  (The squares are powers of two; the
rounding of the one other entry moves the norms' ratio by 3e-8 at most.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import scipy.sparse as sp  # noqa: E402

from paper_1106_3678_amd import binding  # noqa: E402


def test_partial_sums_are_fp64():
    N, slices, wave = 131072, 256, 64
    b = np.zeros(N)
    d = np.ones(N)
    for s in range(slices):
        r = s * 512 + wave * np.arange(8)
        b[r] = 2.0 ** -12
        b[r[0]] = 1.0
        d[r] = 2.0
    f = 5   # a row of the 1s that brings ||b|| to 2^10
    b[f] = np.sqrt(2.0 ** 20 - np.sum(b * b))
    b32 = (b / 2.0 ** 10).astype(np.float32)
    total = np.sum((b32 * b32).astype(np.float64))
    left = np.sum((b32 * b32)[d == 2].astype(np.float64))
    assert left == slices * (2.0 ** -20 + 7 * 2.0 ** -44)
    inner_tol = np.sqrt(left / total) * (1 - 1.0e-7)
    q = np.zeros((N, 1))
    q[f] = 1.0
    x = torch.zeros(N, dtype=torch.float64, device="cuda")
    s = binding.Solver(binding.to_device(sp.diags(d).tocsr()), 1, tol=1e-6, maxit=50,
                       precision=binding.MLB_PREC_FP32_IR, inner_tol=float(inner_tol))
    r = s.solve(torch.from_numpy(b).cuda(), x, binding.column_major(q))
    torch.cuda.synchronize()
    s.close()
    assert r.flag == 0 and r.iter == 1 and r.outer_iters == 1
    assert np.linalg.norm(d * x.cpu().numpy() - b) <= 1e-6 * np.linalg.norm(b)
