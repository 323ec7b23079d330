"""Whole solves in one launch, a group of workgroups per system: sizes at the edges of its slices.

A system of up to 1,048,576 rows (complex and 3x3 blocks 524,288) is solved by P = ceil(N / 512) workgroups, at most
256, each with its own rows (one row a thread in registers up to 512 rows a workgroup, else from
memory).  The sizes below sit at the edges of a wave, of a slice, of the group and of both variants;
the random patterns make every workgroup read rows of every other, with rows of up to 21 entries
(more than one batch of entries).  Against the oracle: the same flag, counts within 5%, x_1..x_20
within 1e-8 relative, the final x within 1e-6 (the bars of the parity tests).  Large systems, which
the oracle takes too long for, are checked by their true residual, and bitwise against a batch of
one, which runs the same kernel from another caller.
"""
import threading

import numpy as np
import pytest
import scipy.sparse as sp

import workloads
from tests.gpu_util import gpu_available, iters_close, rel, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_1106_3678_amd import binding  # noqa: E402


def random_problem(N, per_row, n, seed, cplx=False, bsr=False):
    """Diagonally dominant, entries anywhere in the row."""
    g = np.random.default_rng(seed)
    nb = N // 3 if bsr else N
    k = min(per_row, nb)
    rows = np.repeat(np.arange(nb), k)
    cols = np.concatenate([np.concatenate(([r], g.choice(nb, size=k - 1, replace=False))) for r in range(nb)])
    keep = np.unique(rows * nb + cols, return_index=True)[1]
    rows, cols = rows[keep], cols[keep]
    if bsr:
        v = g.standard_normal((rows.size, 3, 3)) / per_row
        v[rows == cols] += 3.0 * np.eye(3)
        order = np.lexsort((cols, rows))
        rp = np.concatenate(([0], np.cumsum(np.bincount(rows, minlength=nb))))
        A = sp.bsr_matrix((v[order], cols[order].astype(np.int32), rp.astype(np.int32)), shape=(N, N), blocksize=(3, 3))
    else:
        v = g.standard_normal(rows.size) + (1j * g.standard_normal(rows.size) if cplx else 0)
        v = v / np.sqrt(per_row)
        v[rows == cols] += 3.0
        A = sp.csr_matrix((v, (rows, cols)), shape=(N, N))
    b = workloads._gauss(g, N, cplx)
    Q = np.asfortranarray(workloads._gauss(g, (N, n), cplx))
    return workloads.Problem(f"rand{N}_{per_row}_n{n}", A, b, Q, np.zeros(N, dtype=b.dtype), n, 1e-10, 400)


def check(p, precond=0):
    o = run_oracle(p, record=20, precond=precond)
    r, x, its = run_gpu(p, record=20, precond=precond)
    print(f"{p.name}: flag {r.flag}/{o.flag} iter {r.iter}/{o.iter} true {r.err_true:.2e}", flush=True)
    assert r.flag == o.flag == 0
    assert iters_close(r.iter, o.iter)
    for k in range(min(20, o.iter, r.iter)):
        assert rel(its[k], o.x_history[k]) < 1e-8, k + 1
    assert r.err_true < p.tol + 1e-12 and rel(x, o.x) < 1e-6
    _, x2, _ = run_gpu(p, precond=precond)   # without the record
    assert np.array_equal(x, x2)


@pytest.mark.parametrize("N", [1, 63, 64, 65, 511, 512, 513, 1025, 4097])
def test_sizes(N):
    check(random_problem(N, 5, min(4, N), 100 + N))


@pytest.mark.parametrize("n", [1, 3, 4, 5, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("cplx", [False, True])
def test_shadow_counts(n, cplx):
    check(random_problem(1300, 6, n, 300 + n, cplx=cplx))


@pytest.mark.parametrize("per_row", [8, 9, 21])
@pytest.mark.parametrize("cplx", [False, True])
def test_long_rows(per_row, cplx):
    check(random_problem(1111, per_row, 4, 400 + per_row, cplx=cplx))


@pytest.mark.parametrize("N", [3, 510, 513, 1539])
@pytest.mark.parametrize("n", [2, 8, 16])
def test_block_rows(N, n):
    """3x3 blocks; 510 and 1539 rows end a slice inside and between block rows."""
    check(random_problem(N, 7, min(n, N), 500 + N, bsr=True))


def upload(p):
    dA = binding.to_device(p.A)
    return dA, torch.from_numpy(p.b).cuda(), binding.column_major(p.Q)


@pytest.mark.parametrize("m,n", [(362, 2), (363, 4), (512, 1), (724, 4), (1024, 2)])
def test_slices_up_to_the_limit(m, n):
    """131,044, 131,769 (the first past 256 x 512 rows), 262,144, 524,176 and 1,048,576 rows."""
    p = workloads.Problem("sq", workloads.convdiff_2d(m, pe=40.0), None, None, None, n, 1e-8, 20000)
    g = np.random.default_rng(m)
    p.b = p.A @ g.standard_normal(m * m)
    p.Q = np.asfortranarray(g.standard_normal((m * m, n)))
    dA, b, Q = upload(p)
    xs = []
    for batch in (False, True):
        if batch and p.N > 262144:
            break
        x = torch.zeros(p.N, dtype=torch.float64, device="cuda")
        s = binding.Solver(dA, n, tol=p.tol, maxit=p.maxit)
        r = binding.solve_batch([s], [b], [x], [Q])[0] if batch else s.solve(b, x, Q)
        torch.cuda.synchronize()
        xs.append(x.cpu().numpy())
        s.close()
        print(f"m={m} n={n} batch={batch}: iter {r.iter} true {r.err_true:.2e}", flush=True)
        true = np.linalg.norm(p.b - p.A @ xs[-1]) / np.linalg.norm(p.b)
        assert r.flag == 0 and abs(r.err_true - true) < 1e-12 and true < 1e-7
    assert np.array_equal(xs[0], xs[-1])


def test_threads_and_streams():
    """Six threads, each with a stream and a solver of its own, groups that together exceed the device:
    every solve gives bitwise what it gives alone."""
    probs = [workloads.config2(n=4, m=m) for m in (52, 20, 52, 33, 40, 52)]
    data = [upload(p) for p in probs]
    torch.cuda.synchronize()

    def solve(k):
        p, (dA, b, Q) = probs[k], data[k]
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            x = torch.zeros(p.N, dtype=torch.float64, device="cuda")
            s = binding.Solver(dA, p.n, tol=p.tol, maxit=p.maxit, stream=st)
            for _ in range(10):
                x.zero_()
                r = s.solve(b, x, Q)
            st.synchronize()
            s.close()
        return r.flag, r.iter, x.cpu().numpy()

    alone = [solve(k) for k in range(6)]
    got = [None] * 6

    def work(k):
        got[k] = solve(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    for a, b in zip(alone, got):
        assert b is not None and a[:2] == b[:2] and a[0] == 0 and np.array_equal(a[2], b[2])


def test_lost_wait_reports_error(monkeypatch):
    """MLB_GRID_MAX_TRIES=1 makes every wait that is not over at its first look count as lost: the solve
    ends and reports an error, and a new solver runs normally."""
    p = workloads.config2(n=4, m=24)
    dA, b, Q = upload(p)
    x = torch.zeros(p.N, dtype=torch.float64, device="cuda")
    monkeypatch.setenv("MLB_GRID_MAX_TRIES", "1")
    s = binding.Solver(dA, p.n, tol=p.tol, maxit=p.maxit)
    with pytest.raises(binding.MlbError) as e:
        s.solve(b, x, Q)
    assert e.value.code == binding.MLB_EHIP and "gave up" in str(e.value)
    s.close()
    monkeypatch.delenv("MLB_GRID_MAX_TRIES")
    x.zero_()
    s = binding.Solver(dA, p.n, tol=p.tol, maxit=p.maxit)
    assert s.solve(b, x, Q).flag == 0
    s.close()


def test_group_that_leaves_its_gate(monkeypatch):
    """MLB_GRID_ENTRY_TICKS=0: a group that is not complete at once leaves without a result, is started
    again, and after 20 starts the multi-launch iteration solves the system."""
    p = workloads.config2(n=4, m=40)
    dA, b, Q = upload(p)
    monkeypatch.setenv("MLB_GRID_ENTRY_TICKS", "0")
    x = torch.zeros(p.N, dtype=torch.float64, device="cuda")
    s = binding.Solver(dA, p.n, tol=p.tol, maxit=p.maxit)
    r = s.solve(b, x, Q)
    s.close()
    o = run_oracle(p)
    assert r.flag == o.flag == 0 and iters_close(r.iter, o.iter)
    assert rel(x.cpu().numpy(), o.x) < 1e-6 and r.err_true < p.tol + 1e-12
