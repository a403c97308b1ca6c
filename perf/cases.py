"""Timing cases of the multigrid library: the calls that a program makes through
`paper_1208_4247_amd.solver`, over the range of grids, cycles, smoothers and
precisions that the library is used with.

A case is a dict of plain values.  kind:
  solve   Plan.solve from a zero start to a relative residual (the main use)
  vcycle  one V-cycle from zero, the form a preconditioner applies
  fmg     one full-multigrid pass
  batch   BatchPlan.solve of many problems of uneven size
  dst     DstSolver.solve, the exact sine-transform solver
  smooth  Plan.op_smooth on the finest level, for programs that build a cycle
          of their own
Grids have side 2^L - 1 (odd, so rows are never a multiple of a tile or of 16
bytes); `tune` asks for the autotuner, as the benchmark's plans do, and plans
without it run the default tiles, as a plan made with no flags does.
"""
from __future__ import annotations

import math

import torch

from paper_1208_4247_amd import capi
from paper_1208_4247_amd import workloads as wl
from paper_1208_4247_amd.solver import BatchPlan, DstSolver, Plan

DEV = "cuda"


def _solve(name, dim, L, **kw):
    c = dict(kind="solve", dim=dim, L=L, smoother="rbgs", nu1=2, nu2=2, prec="fp64", rhs="noise",
             rtol=1e-10, tune=False)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the benchmark's 2D solve: a few thousand unknowns, where launches and
        # the latency of the coarse levels are all there is
        _solve("solve2d_127", 2, 7, rhs="sine"),
        # a V-cycle from zero on a small 3D grid: the preconditioner call of an
        # outer Krylov loop, enqueued without a wait
        dict(name="vcycle3d_63", kind="vcycle", dim=3, L=6, smoother="rbgs", nu1=2, nu2=2,
             rhs="uniform", tune=False),
        # an ordinary 3D solve with a plan made without flags
        _solve("solve3d_127_v11", 3, 7, nu1=1, nu2=1, rhs="uniform"),
        # the benchmark's 255^3 solves: the default smoother and weighted Jacobi
        _solve("solve3d_255", 3, 8, tune=True),
        _solve("solve3d_255_wj", 3, 8, smoother="wj", tune=True),
        # the benchmark's 511^3 solves, rough data, in both precisions
        _solve("solve3d_511", 3, 9, rhs="uniform", tune=True),
        _solve("solve3d_511_mixed", 3, 9, rhs="uniform", prec="mixed", tune=True),
        # the benchmark's default: about 1.07e9 unknowns, the largest 3D grid
        _solve("solve3d_1023_v11", 3, 10, nu1=1, nu2=1, rhs="modes", tune=True),
        # the benchmark's batch: 128 2D and 128 3D problems, sides 31 .. 1023
        dict(name="batch256", kind="batch", n2d=128, n3d=128, lo2=6, hi2=10, lo3=5, hi3=7,
             nu1=2, nu2=2, smoother="rbgs", graph=True, tune=True),
        # one pass to discretisation accuracy on the largest 2D grid of the paper
        dict(name="fmg2d_4095", kind="fmg", dim=2, L=12, smoother="rbgs", nu1=2, nu2=2,
             rhs="sine", tune=True),
        # the paper's own method: 8-colour Gauss-Seidel, finite-element transfers
        _solve("paper3d_255", 3, 8, smoother="mcgs", nu1=1, nu2=1, rhs="sine", rtol=1e-6),
        # the direct solver that the paper compares full multigrid with
        dict(name="dst3d_255", kind="dst", dim=3, L=8, rhs="noise"),
    ]


def draw(rng):
    kind = rng.choice(["solve"] * 6 + ["vcycle", "fmg", "fmg", "batch", "dst", "smooth"])
    dim = rng.choice([2, 3, 3])
    nu1, nu2 = rng.choice([(1, 1), (1, 2), (2, 1), (2, 2), (2, 3), (3, 3)])
    tune = rng.random() < 0.5
    rhs = rng.choice(["noise", "uniform", "modes", "sine"])
    if kind == "solve":
        form = rng.choice(["rbgs", "rbgs", "rbgs", "mixed", "mixed", "wj", "mcgs"])
        L = rng.randint(4, 11) if dim == 2 else rng.randint(3, 9)
        if dim == 3 and L == 9 and form in ("rbgs", "mixed") and rng.random() < 0.25:
            L, nu1, nu2 = 10, 1, 1
        if form == "mixed" and dim == 3:
            nu1 = min(nu1, 2)
        if form == "mcgs":
            L = min(L, 8 if dim == 3 else 11)
        if form == "wj" and dim == 3:
            L = min(L, 8)
        # the residual's rounding floor grows as (m + 1)^2: no 1e-10 on fine 2D grids
        rtol = rng.choice([1e-6, 1e-8, 1e-10] if L <= 8 or dim == 3 else [1e-6, 1e-7])
        return _solve(None, dim, L, smoother="rbgs" if form == "mixed" else form, nu1=nu1, nu2=nu2,
                      prec="mixed" if form == "mixed" else "fp64", rhs=rhs,
                      rtol=1e-6 if form == "mcgs" else rtol, tune=tune and form != "mcgs")
    if kind == "batch":
        lo2, lo3 = rng.randint(4, 7), rng.randint(3, 5)
        return dict(kind="batch", n2d=rng.randint(1, 90), n3d=rng.randint(1, 70), lo2=lo2,
                    hi2=rng.randint(lo2, 10), lo3=lo3, hi3=rng.randint(lo3, 7), nu1=nu1, nu2=nu2,
                    smoother=rng.choice(["rbgs", "rbgs", "wj"]), graph=rng.random() < 0.7,
                    tune=tune)
    L = rng.randint(5, 12) if dim == 2 else rng.randint(4, 9)
    if kind == "dst":
        return dict(kind="dst", dim=dim, L=L, rhs=rhs)
    if kind == "smooth":
        return dict(kind="smooth", dim=dim, L=L, smoother=rng.choice(["rbgs", "rbgs", "wj"]),
                    nsweeps=rng.randint(1, 4), backward=rng.random() < 0.5,
                    dtype=rng.choice(["f64", "f32"]), rhs=rhs, tune=False)
    return dict(kind=kind, dim=dim, L=L, smoother="rbgs" if kind == "fmg" else
                rng.choice(["rbgs", "rbgs", "wj"]), nu1=nu1, nu2=nu2, rhs=rhs, tune=tune)


# ------------------------------------------------------------------- inputs
def _uniform(shape, seed, stream=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1009 + stream)
    return torch.rand(shape, dtype=torch.float64, device=DEV, generator=g).mul_(2.0).sub_(1.0)


def _rhs(kind, dim, L, seed, stream=0):
    m = (1 << L) - 1
    if kind == "uniform":  # rough data, every frequency
        return _uniform((m,) * dim, seed, stream)
    if kind == "modes":  # a few smooth modes of random amplitude and frequency
        return wl.rhs_sine_modes_device(dim, m, seed, DEV)
    f = wl.sine_product_device(dim, m, DEV).mul_(dim * math.pi ** 2)
    # the model problem, scaled from the seed, or with a little noise
    return f.mul_(1.0 + (seed % 997) / 997.0) if kind == "sine" else \
        f.add_(_uniform((m,) * dim, seed, stream), alpha=1e-3)


def _batch_list(case):
    """(dim, levels) of every problem: sizes cycle through the range unevenly."""
    out = []
    for n, dim, lo, hi in ((case["n2d"], 2, case["lo2"], case["hi2"]),
                           (case["n3d"], 3, case["lo3"], case["hi3"])):
        out += [(dim, lo + int(k)) for k in (wl.uniform_int(4, dim, n, 0, hi - lo) if n else [])]
    return out


def _grids(probs):
    """One allocation for the grids of a batch, and a view of each in it (every
    grid starts at a multiple of 512 bytes; the gaps hold zeros)."""
    sizes = [((1 << L) - 1) ** d for d, L in probs]
    at = [0]
    for n in sizes:
        at.append(at[-1] + -(-n // 64) * 64)
    flat = torch.zeros(at[-1], dtype=torch.float64, device=DEV)
    return flat, [flat[a:a + n].view((((1 << L) - 1),) * d)
                  for a, n, (d, L) in zip(at, sizes, probs)]


def _batch_rhs(probs, seed):
    flat, fs = _grids(probs)
    for q, f in enumerate(fs):
        f.copy_(_uniform(tuple(f.shape), seed, 1 + q))
    return flat, fs


def _plan(case, **kw):
    flags = (capi.GMG_AUTOTUNE if case["tune"] else 0) | \
        (capi.GMG_FE_TRANSFER if case["smoother"] == "mcgs" else 0)
    return Plan(case["dim"], case["L"], smoother=case["smoother"], flags=flags, **kw)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        probs = _batch_list(case)
        _, fs = _batch_rhs(probs, seed)
        flat, us = _grids(probs)
        flags = (capi.GMG_USE_GRAPH if case["graph"] else 0) | \
            (capi.GMG_AUTOTUNE if case["tune"] else 0)
        plan = BatchPlan(probs, smoother=case["smoother"], nu1=case["nu1"], nu2=case["nu2"],
                         flags=flags)
        return dict(case=case, plan=plan, f=fs, u=us, flat=flat)
    f = _rhs(case["rhs"], case["dim"], case["L"], seed)
    if kind == "dst":
        return dict(case=case, plan=DstSolver(case["dim"], case["L"]), f=f, u=torch.empty_like(f))
    if kind == "smooth":
        dt = torch.float32 if case["dtype"] == "f32" else torch.float64
        start = _uniform(tuple(f.shape), seed, 7).to(dt)
        plan = _plan(case, precision="mixed" if dt == torch.float32 else "fp64")
        return dict(case=case, plan=plan, f=f.to(dt), start=start, u=torch.empty_like(start))
    plan = _plan(case, nu1=case["nu1"], nu2=case["nu2"], precision=case.get("prec", "fp64"))
    return dict(case=case, plan=plan, f=f, u=torch.zeros_like(f))


def run(state):
    case, plan, f, u = state["case"], state["plan"], state["f"], state["u"]
    kind = case["kind"]
    if kind == "solve":
        u.zero_()
        _, iters, relres = plan.solve(u, f, rtol=case["rtol"])
        return dict(u=u, iters=iters, relres=relres)
    if kind == "vcycle":
        u.zero_()
        plan.vcycle(u, f)
        return dict(u=u)
    if kind == "batch":
        state["flat"].zero_()
        _, iters, relres, _ = plan.solve(u, f, rtol=1e-10)
        return dict(u=state["flat"], iters=torch.tensor(iters), relres=torch.tensor(relres))
    if kind == "fmg":
        plan.fmg(u, f)
    elif kind == "dst":
        plan.solve(u, f)
    else:
        plan.op_smooth(0, case["nsweeps"], case["backward"], state["start"], f, None, u)
    return dict(u=u)


# --------------------------------------------------------------------- work
def _hier(dim, L):
    """Unknowns of all levels of the hierarchy."""
    return sum(((1 << k) - 1) ** dim for k in range(1, L + 1))


def _cycles(case):
    """Cycles to the tolerance, from the smoother's contraction per cycle."""
    nu = min(case["nu1"] + case["nu2"], 6)
    rho = {"rbgs": {2: 0.42, 3: 0.27, 4: 0.17, 5: 0.14, 6: 0.12},
           "wj": {2: 0.60, 3: 0.48, 4: 0.33, 5: 0.28, 6: 0.24},
           "mcgs": {2: 0.38, 3: 0.28, 4: 0.22, 5: 0.18, 6: 0.15}}[case["smoother"]][nu]
    return math.ceil(math.log(case.get("rtol", 1e-10)) / math.log(rho))


def work(case):
    """Bytes: f read and u read and written once for each V-cycle on every
    level (a cycle smooths the iterate that the one before left); one pass over
    the arrays for the rest.  Flops: 2d + 3 for an update or a residual."""
    kind = case["kind"]
    if kind == "batch":
        n = sum(_hier(d, L) for d, L in _batch_list(case))
        k, d = _cycles(case), 3
        return dict(bytes=24.0 * n * k, flops=(2 * d + 3.0) * n * k * (case["nu1"] + case["nu2"] + 1))
    d, L = case["dim"], case["L"]
    n0 = ((1 << L) - 1) ** d
    if kind == "smooth":
        w = 4 if case["dtype"] == "f32" else 8
        return dict(bytes=3.0 * w * n0, flops=(2 * d + 3.0) * n0 * case["nsweeps"])
    if kind == "dst":
        return dict(bytes=16.0 * n0, flops=2.0 * d * 5.0 * n0 * (L + 1))
    n = _hier(d, L)
    ops = (2 * d + 3.0) * (case["nu1"] + case["nu2"] + 1)
    if kind == "vcycle":
        return dict(bytes=16.0 * n0, flops=ops * n)
    if kind == "fmg":  # one V-cycle from each level down
        return dict(bytes=16.0 * n0, flops=ops * n * 2 ** d / (2 ** d - 1.0))
    k = _cycles(case)
    return dict(bytes=(12.0 if case["prec"] == "mixed" else 24.0) * n * k, flops=ops * n * k)


# -------------------------------------------------------------------- exact
def _direct(f):
    """A^-1 f by dense sine matrices along every axis."""
    m, d = f.shape[0], f.dim()
    n = m + 1
    k = torch.arange(1, n, device=DEV)
    s = torch.sin((torch.outer(k, k) % (2 * n)).double() * (math.pi / n)) * math.sqrt(2.0 / n)
    lam = (2.0 * n * torch.sin(k.double() * (math.pi / (2 * n)))) ** 2

    def along_all(x):
        for _ in range(d):  # the last axis, then rotated to the front
            x = (x.reshape(-1, m) @ s).reshape(x.shape).movedim(-1, 0).contiguous()
        return x

    x = along_all(f)
    for a in range(d):
        part = lam.reshape([m if b == a else 1 for b in range(d)])
        total = part if a == 0 else total + part
    return along_all(x.div_(total))


def _pad(u):
    return torch.nn.functional.pad(u, (1, 1) * u.dim())


def _nbsum(u):
    p, m, d = _pad(u), u.shape[0], u.dim()
    total = torch.zeros_like(u)
    for a in range(d):
        for s in (0, 2):
            total += p[tuple(slice(s, s + m) if b == a else slice(1, 1 + m) for b in range(d))]
    return total


def _red(u):
    i = torch.arange(1, u.shape[0] + 1, device=DEV)
    total = sum(i.reshape([-1 if b == a else 1 for b in range(u.dim())]) for a in range(u.dim()))
    return total % 2 == 0


def _sweeps(u, f, smoother, count, backward):
    d, n = u.dim(), u.shape[0] + 1
    if smoother == "wj":
        om = 2.0 * d / (2 * d + 1)
        for _ in range(count):
            u = (1 - om) * u + om * (f / n ** 2 + _nbsum(u)) / (2 * d)
        return u
    red = _red(u)
    for _ in range(count):
        for colour in ((~red, red) if backward else (red, ~red)):
            u = torch.where(colour, (f / n ** 2 + _nbsum(u)) / (2 * d), u)
    return u


def _down(r):
    """Full weighting."""
    for a in range(r.dim()):
        k = r.shape[a]
        r = 0.5 * r.narrow(a, 1, k - 2) + 0.25 * (r.narrow(a, 0, k - 2) + r.narrow(a, 2, k - 2))
        r = r.index_select(a, torch.arange(0, k - 2, 2, device=DEV))
    return r


def _up(e):
    """(Bi/tri)linear interpolation."""
    for a in range(e.dim()):
        k = e.shape[a]
        x = torch.zeros([2 * k + 1 if b == a else s for b, s in enumerate(e.shape)],
                        dtype=e.dtype, device=e.device)
        at = torch.arange(k, device=DEV)
        x.index_add_(a, 2 * at + 1, e)
        x.index_add_(a, 2 * at, 0.5 * e)
        x.index_add_(a, 2 * at + 2, 0.5 * e)
        e = x
    return e


def _vcycle(u, f, case):
    d, n = f.dim(), f.shape[0] + 1
    if n == 2:
        return f / n ** 2 / (2 * d)
    u = _sweeps(u, f, case["smoother"], case["nu1"], False)
    fc = _down(f - (2 * d * u - _nbsum(u)) * n ** 2)
    u = u + _up(_vcycle(torch.zeros_like(fc), fc, case))
    return _sweeps(u, f, case["smoother"], case["nu2"], True)


def _fmg(f, case):
    if f.shape[0] == 1:
        return f / 4 / (2 * f.dim())
    return _vcycle(_up(_fmg(_down(f), case)), f, case)


def exact(case, seed):
    """In 64 bits with torch's own operations: the solution of the linear system
    for the solvers, the cycle written out for the rest."""
    kind = case["kind"]
    if kind == "batch":
        flat, fs = _batch_rhs(_batch_list(case), seed)
        for f in fs:
            f.copy_(_direct(f))
        return dict(u=flat, iters=None, relres=None)
    f = _rhs(case["rhs"], case["dim"], case["L"], seed)
    if kind == "smooth":
        dt = torch.float32 if case["dtype"] == "f32" else torch.float64
        start = _uniform(tuple(f.shape), seed, 7).to(dt).double()
        return dict(u=_sweeps(start, f.to(dt).double(), case["smoother"], case["nsweeps"],
                              case["backward"]))
    if kind == "vcycle":
        return dict(u=_vcycle(torch.zeros_like(f), f, case))
    if kind == "fmg":
        return dict(u=_fmg(f, case))
    u = _direct(f)
    return dict(u=u) if kind == "dst" else dict(u=u, iters=None, relres=None)
