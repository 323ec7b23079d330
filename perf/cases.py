"""The solves this library is timed on: complete calls of its public entry points (paper_1106_3678_amd.binding).

Every system is built on the GPU from a seed: convection-diffusion on a square or a cube (first-order upwind,
constant velocity), a complex shifted Helmholtz operator with convection, or a reservoir-shaped 3x3-block system.
The right-hand side is A x_true for a smooth x_true (a few low sine modes, as the fields such discretisations
are solved for), so that the exact solution is known; Q is standard normal, as the method asks for.

A case is a dict of plain values:
  entry    solve   one right-hand side on a prepared solver (the usual call; the matrix stays, b is new)
           batch   `count` prepared small systems in one launch
           server  `count` requests of uneven size submitted at once and collected
           once    the allocation-free call: A^H, workspace and solve of a matrix not seen before
  system   convdiff2d, convdiff3d, helmholtz3d (m points a side) or reservoir (nx x ny x nz cells)
  n, tol, precond (none, jacobi, ilu0), ir (fp32 inner iteration), tf (transpose-free)
"""
import math
import random

import torch

from paper_1106_3678_amd import binding

PRECOND = {"none": binding.MLB_PRECOND_NONE, "jacobi": binding.MLB_PRECOND_JACOBI, "ilu0": binding.MLB_PRECOND_ILU0}
MAXIT = 20000
DEV = "cuda"


def _case(entry, system, n, tol=1e-11, pe=0.0, precond="none", ir=False, tf=False, **size):
    return dict(entry=entry, system=system, n=n, tol=tol, pe=pe, precond=precond, ir=ir, tf=tf, **size)


def listed():
    return [
        # the smallest solve: the 32 x 32 square of the smoke test and the parity tests; bound by latency
        dict(name="square_32", **_case("solve", "convdiff2d", 4, pe=5.0, m=32)),
        # an ordinary 2D solve of ragged size (32,761 rows), the middle of the serving trace's range
        dict(name="square_181", **_case("solve", "convdiff2d", 2, pe=12.0, m=181)),
        # an ordinary 3D solve of ragged size (103,823 rows) with more shadow vectors
        dict(name="cube_47", **_case("solve", "convdiff3d", 8, pe=20.0, m=47)),
        # the benchmark's default system
        dict(name="cube_128", **_case("solve", "convdiff3d", 4, pe=20.0, m=128)),
        # the benchmark's complex system: complex values, many shadow vectors
        dict(name="helmholtz_96", **_case("solve", "helmholtz3d", 16, pe=10.0, m=96)),
        # the benchmark's 3x3-block system at full size with block Jacobi; an accumulation term as of a short
        # time step, where such a simulator calls the solver
        dict(name="reservoir_jacobi", **_case("solve", "reservoir", 8, precond="jacobi", nx=60, ny=220, nz=85)),
        # ILU(0), the preconditioner of the paper's experiments, on a cube and on a block system
        dict(name="cube_96_ilu0", **_case("solve", "convdiff3d", 4, pe=20.0, precond="ilu0", m=96)),
        dict(name="reservoir_ilu0", **_case("solve", "reservoir", 4, precond="ilu0", nx=31, ny=57, nz=24)),
        # fp32 inner iteration with fp64 refinement
        dict(name="cube_64_ir", **_case("solve", "convdiff3d", 4, pe=20.0, ir=True, m=64)),
        # 64 small systems in one launch, one workgroup each (16 to 48 points a side)
        dict(name="batch_64", **_case("batch", "convdiff2d", 4, pe=5.0, m=32, count=64)),
        # requests of uneven size (1e3 to 3e5 rows, 2D and 3D) submitted at once, as a server under load has them
        dict(name="server_24", **_case("server", "convdiff3d", 4, pe=20.0, m=40, count=24)),
        # a matrix not seen before in a caller that cannot allocate, without A^H
        dict(name="once_33_tf", **_case("once", "convdiff3d", 4, pe=20.0, tf=True, m=33)),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    kind = rng.choice(["2d", "3d", "3d", "helmholtz", "reservoir", "ilu3d", "ilures", "ir", "batch", "server", "once"])
    n = rng.choice([1, 2, 3, 4, 4, 5, 8])
    pe = round(math.exp(rng.uniform(math.log(2.0), math.log(40.0))), 3)
    if kind == "2d":
        return _case("solve", "convdiff2d", n, pe=pe, m=_log(rng, 20, 500))
    if kind == "3d":
        return _case("solve", "convdiff3d", rng.choice([1, 2, 3, 4, 6, 8, 12, 16]), pe=pe, m=_log(rng, 10, 128),
                     tf=rng.random() < 0.2)
    if kind == "helmholtz":
        return _case("solve", "helmholtz3d", rng.choice([2, 4, 7, 8, 16]), pe=round(rng.uniform(5.0, 20.0), 3),
                     m=_log(rng, 12, 96))
    if kind in ("reservoir", "ilures"):
        big = kind == "reservoir"
        return _case("solve", "reservoir", rng.choice([2, 4, 8]), precond="jacobi" if big else "ilu0",
                     nx=_log(rng, 10, 60 if big else 40), ny=_log(rng, 10, 220 if big else 60),
                     nz=_log(rng, 5, 85 if big else 30))
    if kind == "ilu3d":
        return _case("solve", "convdiff3d", rng.choice([1, 2, 4, 8]), pe=pe, precond="ilu0", m=_log(rng, 10, 96))
    if kind == "ir":
        return _case("solve", "convdiff3d", n, pe=pe, ir=True, m=_log(rng, 16, 80))
    if kind == "batch":
        return _case("batch", "convdiff2d", n, pe=pe, m=_log(rng, 16, 48), count=_log(rng, 8, 128))
    if kind == "server":
        return _case("server", "convdiff3d", n, pe=pe, m=40, count=_log(rng, 4, 32))
    return _case("once", rng.choice(["convdiff2d", "convdiff3d"]), rng.choice([2, 3, 4]), pe=pe, m=_log(rng, 12, 48),
                 tf=rng.random() < 0.5)


# ---- systems --------------------------------------------------------------------------------------------------


def _neighbours(shape):
    """Cell numbers (x fastest) and, for each of the 2d + 1 stencil points in column order, (axis, step, mask, column).
    `shape` is (.., ny, nx)."""
    d = len(shape)
    cells = torch.arange(math.prod(shape), device=DEV).reshape(shape)
    points = []
    for axis in range(d):
        for step in (-1, 1):
            size = shape[axis]
            pos = torch.arange(size, device=DEV).reshape([-1 if a == axis else 1 for a in range(d)]).expand(shape)
            inside = (pos > 0) if step < 0 else (pos < size - 1)
            points.append((axis, step, inside.reshape(-1), (cells + step * math.prod(shape[axis + 1:])).reshape(-1)))
    points.append((-1, 0, torch.ones(cells.numel(), dtype=torch.bool, device=DEV), cells.reshape(-1)))
    rank = {p: (p[1] * (d - p[0]) if p[0] >= 0 else 0) for p in [(q[0], q[1]) for q in points]}
    return sorted(points, key=lambda p: rank[(p[0], p[1])])


def _modes(shape, host, cplx):
    """A smooth field: random low sine modes that vanish outside the grid."""
    total = None
    for _ in range(3):
        term = None
        for size in shape:
            k = host.randint(1, 3)
            s = torch.sin(math.pi * k * (torch.arange(size, device=DEV, dtype=torch.float64) + 1) / (size + 1))
            term = s if term is None else term.unsqueeze(-1) * s
        amp = complex(host.gauss(0, 1), host.gauss(0, 1)) if cplx else host.gauss(0, 1)
        total = amp * term if total is None else total + amp * term
    return total.reshape(-1)


def _smooth_noise(shape, sigma, gen):
    """White noise after a periodic Gaussian filter of `sigma` cells, unit variance."""
    z = torch.randn(shape, dtype=torch.float64, device=DEV, generator=gen)
    f = torch.fft.fftn(z)
    for axis, size in enumerate(shape):
        k = torch.fft.fftfreq(size, device=DEV, dtype=torch.float64)
        f = f * torch.exp(-2.0 * (math.pi * sigma * k) ** 2).reshape([-1 if a == axis else 1 for a in range(len(shape))])
    z = torch.fft.ifftn(f).real
    return (z - z.mean()) / z.std()


def _shape(case):
    if case["system"] == "reservoir":
        return (case["nz"], case["ny"], case["nx"])
    return (case["m"],) * (2 if case["system"].endswith("2d") else 3)


def _x_true(case, seed):
    host = random.Random(seed)
    shape = _shape(case)
    if case["system"] == "reservoir":
        return torch.stack([_modes(shape, host, False) for _ in range(3)], 1).reshape(-1).contiguous()
    return _modes(shape, host, case["system"] == "helmholtz3d")


def _grid_matrix(case, seed):
    """(DeviceMatrix, product) of a scalar stencil, multiplied by h^2: per axis 2 + 2 Pe |v| on the diagonal,
    -1 - 2 Pe |v| on the upwind and -1 on the downwind neighbour."""
    host = random.Random(seed + 1)
    shape = _shape(case)
    v = [host.gauss(0, 1) for _ in shape]
    norm = math.sqrt(sum(a * a for a in v))
    v = [2.0 * case["pe"] * a / norm for a in v]
    diag = sum(2.0 + abs(a) for a in v)
    cplx = case["system"] == "helmholtz3d"
    if cplx:
        diag = diag - (10.0 / (case["m"] + 1)) ** 2 * (1.0 - 0.5j)
    vals, mask, cols = [], [], []
    for axis, step, inside, col in _neighbours(shape):
        value = diag if axis < 0 else -1.0 - (abs(v[axis]) if v[axis] * step < 0 else 0.0)
        vals.append(value)
        mask.append(inside)
        cols.append(col)
    mask, cols = torch.stack(mask, 1), torch.stack(cols, 1)
    N = mask.shape[0]
    dt = torch.complex128 if cplx else torch.float64
    full = torch.tensor(vals, dtype=dt, device=DEV).expand(N, -1)
    rp = torch.zeros(N + 1, dtype=torch.int32, device=DEV)
    rp[1:] = mask.sum(1).cumsum(0)
    A = binding.DeviceMatrix(rp, cols[mask].to(torch.int32), full[mask].contiguous(), N, binding.MLB_CSR,
                             binding.MLB_C128 if cplx else binding.MLB_R64)
    safe = torch.where(mask, cols, 0)

    def product(x):
        return torch.where(mask, full * x[safe], 0).sum(1)
    return A, product


def _reservoir_matrix(case, seed):
    """(DeviceMatrix, product) of a 7-point 3x3-block system: log-normal permeability (smoothed over 8 cells), face
    transmissibilities by harmonic means, one-sided coupling along a potential, an accumulation term."""
    shape = _shape(case)
    gen = torch.Generator(device=DEV).manual_seed(seed + 1)
    K = torch.exp(1.0 * _smooth_noise(shape, 8.0 / math.sqrt(2.0), gen)).reshape(-1)
    pot = _smooth_noise(shape, 8.0, gen)
    pot = (pot + torch.linspace(0, 4, shape[2], device=DEV, dtype=torch.float64)).reshape(-1)
    C = torch.eye(3, dtype=torch.float64, device=DEV) + 0.1 * torch.randn(3, 3, dtype=torch.float64, device=DEV, generator=gen)
    U = 0.5 * torch.randn(3, 3, dtype=torch.float64, device=DEV, generator=gen).abs()
    points = _neighbours(shape)
    ncell = K.numel()
    blocks, diag, tsum, count = [], 0, 0, 0
    for axis, step, inside, col in points:
        if axis < 0:
            blocks.append(None)
            continue
        at = torch.where(inside, col, 0)
        T = torch.where(inside, 2.0 * K * K[at] / (K + K[at]), 0)
        theta = (pot[at] > pot).to(torch.float64)
        blk = T[:, None, None] * (C + theta[:, None, None] * U)
        blocks.append(-blk)
        diag = diag + blk
        tsum, count = tsum + T, count + inside
    diag = diag + (0.5 * tsum / count + 1e-3)[:, None, None] * torch.eye(3, dtype=torch.float64, device=DEV)
    blocks = torch.stack([diag if b is None else b for b in blocks], 1)
    mask, cols = torch.stack([p[2] for p in points], 1), torch.stack([p[3] for p in points], 1)
    rp = torch.zeros(ncell + 1, dtype=torch.int32, device=DEV)
    rp[1:] = mask.sum(1).cumsum(0)
    A = binding.DeviceMatrix(rp, cols[mask].to(torch.int32), blocks[mask].reshape(-1), 3 * ncell, binding.MLB_BSR3,
                             binding.MLB_R64)

    def product(x):
        x = x.reshape(-1, 3)
        y = torch.zeros_like(x)
        for k in range(mask.shape[1]):
            at = torch.where(mask[:, k], cols[:, k], 0)
            y += (blocks[:, k] * torch.where(mask[:, k, None], x[at], 0)[:, None, :]).sum(2)
        return y.reshape(-1)

    return A, product


def _system(case, seed):
    """One linear system with what a program keeps for it: (A, b, x, Q)."""
    A, product = (_reservoir_matrix if case["system"] == "reservoir" else _grid_matrix)(case, seed)
    b = product(_x_true(case, seed)).contiguous()
    gen = torch.Generator(device=DEV).manual_seed(seed + 2)
    Q = torch.randn((case["n"], A.nrows), dtype=b.dtype, device=DEV, generator=gen).t()
    return A, b, torch.zeros_like(b), Q


def _members(case):
    """The systems of a batch or of a server's load: uneven sizes, the same for every seed."""
    rng = random.Random(case["count"])
    out = []
    for _ in range(case["count"]):
        c = dict(case)
        if case["entry"] == "batch":
            c["m"] = rng.randint(max(8, case["m"] // 2), case["m"] * 3 // 2)
        else:
            two = rng.random() < 0.5
            c["system"] = "convdiff2d" if two else "convdiff3d"
            c["m"] = int(round(math.exp(rng.uniform(math.log(1e3), math.log(3e5))) ** (0.5 if two else 1 / 3)))
            c["n"] = rng.choice([2, 4, 8])
            c["pe"] = case["pe"] * rng.uniform(0.5, 2.0)
        out.append(c)
    return out


# ---- the calls ------------------------------------------------------------------------------------------------


def _solver(case, A):
    return binding.Solver(A, case["n"], tol=case["tol"], maxit=MAXIT, precond=PRECOND[case["precond"]],
                          precision=binding.MLB_PREC_FP32_IR if case["ir"] else binding.MLB_PREC_FP64,
                          transpose_free=case["tf"])


def prepare(case, seed):
    if case["entry"] in ("solve", "once"):
        A, b, x, Q = _system(case, seed)
        return dict(case=case, A=A, b=b, x=x, Q=Q, solver=_solver(case, A) if case["entry"] == "solve" else None)
    cases = _members(case)
    systems = [_system(c, seed + 7 * k) for k, c in enumerate(cases)]
    x = torch.cat([s[2] for s in systems])
    xs = list(x.split([s[2].numel() for s in systems]))
    state = dict(case=case, cases=cases, A=[s[0] for s in systems], b=[s[1] for s in systems], x=x, xs=xs,
                 Q=[s[3] for s in systems])
    if case["entry"] == "batch":
        state["solvers"] = [_solver(c, A) for c, A in zip(cases, state["A"])]
    else:
        state["server"] = binding.Server(64 << 30, 8)
    return state


def run(state):
    case, x = state["case"], state["x"]
    x.zero_()   # the initial guess
    if case["entry"] == "solve":
        r = state["solver"].solve(state["b"], x, state["Q"])
        return dict(x=x, flag=r.flag)
    if case["entry"] == "once":
        r = binding.solve_noalloc(state["A"], state["b"], x, state["Q"], case["n"], tol=case["tol"], maxit=MAXIT,
                                  transpose_free=case["tf"])
        return dict(x=x, flag=r.flag)
    if case["entry"] == "batch":
        rs = binding.solve_batch(state["solvers"], state["b"], state["xs"], state["Q"])
        return dict(x=x, flag=sum(abs(r.flag) for r in rs))
    torch.cuda.synchronize()   # the server's streams do not wait for the caller's
    server = state["server"]
    tickets = [server.submit(A, b, xk, Q, c["n"], tol=c["tol"], maxit=MAXIT)
               for c, A, b, xk, Q in zip(state["cases"], state["A"], state["b"], state["xs"], state["Q"])]
    rs = [server.wait(t)[0] for t in tickets]
    return dict(x=x, flag=sum(abs(r.flag) for r in rs))


def exact(case, seed):
    if case["entry"] in ("solve", "once"):
        return dict(x=_x_true(case, seed), flag=None)
    return dict(x=torch.cat([_x_true(c, seed + 7 * k) for k, c in enumerate(_members(case))]), flag=None)


# ---- what a call cannot do without ----------------------------------------------------------------------------


def _iterations(case):
    """About how many iterations a solve of this size takes (measured over the ranges of draw())."""
    if case["system"] == "reservoir":
        return 25 if case["precond"] == "ilu0" else 100
    m = case["m"]
    k = {"convdiff2d": 15 + 1.4 * m, "convdiff3d": 20 + 1.85 * m, "helmholtz3d": 15 + 2.0 * m}[case["system"]]
    return 10 + 0.45 * m if case["precond"] == "ilu0" else 2.5 * k if case["ir"] else k


def _work(case):
    """An iteration multiplies by A 1 + 1/n times and takes part of it through the n-column blocks W, G, Q and F (A^H Q;
    none without A^H) and the residual: each of these read once, w, g, r and x written once."""
    cells = math.prod(_shape(case))
    rows = 3 * cells if case["system"] == "reservoir" else cells
    entry = 9 if case["system"] == "reservoir" else 1
    points = 2 * len(_shape(case)) + 1
    size = 16 if case["system"] == "helmholtz3d" else 4 if case["ir"] else 8
    n, its = case["n"], _iterations(case)
    matrix = points * cells * (entry * size + 4) * (2 if case["precond"] == "ilu0" else 1)   # and the two factors
    flop = 8 if case["system"] == "helmholtz3d" else 2
    return dict(bytes=its * ((1 + 1 / n) * matrix + (2.5 * n + 5) * rows * size),
                flops=its * ((1 + 1 / n) * points * cells * entry * (2 if case["precond"] == "ilu0" else 1) +
                             (5 * n + 4) * rows) * flop)


def work(case):
    parts = [_work(c) for c in (_members(case) if case["entry"] in ("batch", "server") else [case])]
    return {k: float(sum(p[k] for p in parts)) for k in ("bytes", "flops")}
