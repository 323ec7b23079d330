"""A solve on a stream that still holds earlier work does not keep another thread's solve waiting for that
work: the two groups together exceed the card, and the second one ends while the first one's stream is busy."""
import threading

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import workloads  # noqa: E402
from paper_1106_3678_amd import binding  # noqa: E402


def system(m, stream=None):
    A = workloads.convdiff_2d(m, pe=5.0)
    g = np.random.default_rng(m)
    b = torch.from_numpy(g.standard_normal(m * m)).cuda()
    Q = binding.column_major(g.standard_normal((m * m, 2)))
    return binding.Solver(binding.to_device(A), 2, tol=1e-3, maxit=2000, stream=stream), b, torch.zeros_like(b), Q


def test_busy_stream_holds_nobody_up():
    st = torch.cuda.Stream()
    first = system(250, st)    # 62,500 rows: 123 slices, on a stream of its own
    second = system(320)       # 102,400 rows: 200 slices, on the default stream
    w = torch.randn(4096, 4096, device="cuda")
    out = torch.empty_like(w)
    for s, b, x, Q in (first, second):   # first use of the kernels
        s.solve(b, x, Q)
        x.zero_()
    torch.mm(w, w, out=out)
    torch.cuda.synchronize()
    t0, t1, busy = (torch.cuda.Event(enable_timing=True) for _ in range(3))
    t0.record()
    torch.mm(w, w, out=out)
    t1.record()
    torch.cuda.synchronize()
    count = int(min(4000, max(50, 500.0 / t0.elapsed_time(t1))))   # about half a second
    flags = {}

    def solve_first():
        s, b, x, Q = first
        flags["first"] = s.solve(b, x, Q).flag

    with torch.cuda.stream(st):
        for _ in range(count):
            torch.mm(w, w, out=out)
        busy.record()
    t = threading.Thread(target=solve_first)
    t.start()
    t.join(0.05)               # it has its stream's work before it
    assert not busy.query()
    s, b, x, Q = second
    flags["second"] = s.solve(b, x, Q).flag
    early = not busy.query()
    t.join()
    torch.cuda.synchronize()
    for s in (first[0], second[0]):
        s.close()
    assert flags == {"first": 0, "second": 0} and early
