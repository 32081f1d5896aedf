"""The workloads by which this library's speed is followed.

Each case is one call (or one training step) that a program makes through the
public entry points: whole solves from the smallest grid of the named
workloads to one GPU's full share, batched solves, the differentiable solve
with its gradients, and the single blocks of the preconditioner and the
operator (V-cycle, smoother, SpMV), single and batched, in every storage
precision.  `exact` evaluates the same inputs in FP64 with plain torch.

Solves run to a residual of 1e-11 (where x is the solution to FP64 accuracy
whatever the rounding of the inner steps) or, on the large grids, for one
restart cycle of a fixed number of steps, which is what a timed phase of the
benchmark repeats.
"""
import math

import torch

from paper_2507_11512_amd import hpgmx
from paper_2507_11512_amd.autograd import StencilSolver

DTYPE = {"fp64": hpgmx.F64, "fp32": hpgmx.F32, "fp16": hpgmx.F16, "bf16": hpgmx.BF16,
         "fp16-mg": hpgmx.F16_MG, "bf16-mg": hpgmx.BF16_MG}
VEC = {"fp64": torch.float64, "fp16-mg": torch.float16, "bf16-mg": torch.bfloat16}
SWEEP = {"forward": hpgmx.GS_FORWARD, "backward": hpgmx.GS_BACKWARD, "symmetric": hpgmx.GS_SYMMETRIC}
TOL = 1e-11
RESTART = 30
BETA = 0.5


def listed():
    return [
        # The smallest named workload: 4096 unknowns, symmetric sweeps; launches and latency are all of it.
        dict(name="solve-16", kind="solve", nx=16, ny=16, nz=16, levels=3, sweep="symmetric", inner="fp32",
             cols="int32", nrhs=1, steps=0),
        # An ordinary small solve on a grid that is no cube, matrices held in binary16.
        dict(name="solve-48x40x32-fp16", kind="solve", nx=48, ny=40, nz=32, levels=3, sweep="forward",
             inner="fp16", cols="int32", nrhs=1, steps=0),
        # The middle workload: 2.1M unknowns, to convergence.
        dict(name="solve-128", kind="solve", nx=128, ny=128, nz=128, levels=4, sweep="forward", inner="fp32",
             cols="int32", nrhs=1, steps=0),
        # One GPU's full share (32.8M unknowns): one restart cycle.
        dict(name="solve-320", kind="solve", nx=320, ny=320, nz=320, levels=4, sweep="forward", inner="fp32",
             cols="int32", nrhs=1, steps=30),
        # The all-FP64 solver that every mixed-precision result is validated against: one restart cycle.
        dict(name="solve-fp64-192x176x160", kind="solve", nx=192, ny=176, nz=160, levels=4, sweep="forward",
             inner="fp64", cols="int32", nrhs=1, steps=30),
        # Eight right-hand sides at once, the batched workload: one restart cycle.
        dict(name="batch-8x192", kind="solve", nx=192, ny=192, nz=192, levels=4, sweep="forward", inner="fp32",
             cols="int32", nrhs=8, steps=30),
        # A few right-hand sides on a small ragged grid (padded to a batch of four), to convergence.
        dict(name="batch-3x40x48x56", kind="solve", nx=40, ny=48, nz=56, levels=4, sweep="forward", inner="fp32",
             cols="int32", nrhs=3, steps=0),
        # The preconditioner alone, whole hierarchy in bfloat16, at the low-precision workload's size.
        dict(name="vcycle-256-bf16", kind="vcycle", nx=256, ny=256, nz=256, levels=4, sweep="forward",
             inner="bf16-mg", cols="int32", nrhs=1),
        # The preconditioner alone in FP32 with symmetric sweeps, levels with odd extents.
        dict(name="vcycle-200x152x104-sym", kind="vcycle", nx=200, ny=152, nz=104, levels=4, sweep="symmetric",
             inner="fp32", cols="int32", nrhs=1),
        # One smoother sweep from a given start in FP64 on a grid with odd extents.
        dict(name="smooth-149x101x83-fp64", kind="smooth", nx=149, ny=101, nz=83, levels=1, sweep="backward",
             inner="fp64", cols="int32", nrhs=1),
        # One product with the operator, 16-bit column offsets.
        dict(name="spmv-256x224x240-offset16", kind="spmv", nx=256, ny=224, nz=240, levels=2, sweep="forward",
             inner="fp32", cols="offset16", nrhs=1),
        # One training step through the solver: two right-hand sides, gradients of b and of the 27 stencil entries.
        dict(name="adjoint-2x24x20x16", kind="adjoint", nx=24, ny=20, nz=16, levels=3, sweep="forward",
             inner="fp32", cols="int32", nrhs=2, steps=0),
    ]


def _extents(rng, levels, lo, hi, even):
    """Three extents divisible by 2^(levels-1) (twice that if the coarsest level is to be even too), with a mean
    edge between lo and hi."""
    f = 1 << (levels - 1 + (1 if even else 0))
    edge = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    out = []
    for _ in range(3):
        n = max(2 if even else 1, round(edge * rng.uniform(0.75, 1.25) / f)) * f
        out.append(max(n, 2 * (1 << (levels - 1))))
    return out


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "batch", "batch", "vcycle", "vcycle", "smooth", "spmv", "adjoint"])
    c = {}
    if kind == "solve":
        large = rng.random() < 0.4
        levels = 4 if large else rng.choice([2, 3, 3, 4])
        nx, ny, nz = _extents(rng, levels, 128 if large else 14, 180 if large else 88, rng.random() < 0.7)
        inner = rng.choice(["fp32", "fp32", "fp64", "fp16", "bf16"])
        c = dict(kind="solve", inner=inner, nrhs=1, steps=rng.choice([20, 30]) if large else 0,
                 cols=rng.choice(["int32", "int32", "offset16"]))
    elif kind == "batch":
        large = rng.random() < 0.4
        levels = 4 if large else rng.choice([2, 3, 4])
        nx, ny, nz = _extents(rng, levels, 72 if large else 14, 112 if large else 56, rng.random() < 0.7)
        c = dict(kind="solve", inner=rng.choice(["fp32", "fp32", "fp64", "fp16"]), nrhs=rng.randint(2, 8),
                 steps=rng.choice([20, 30]) if large else 0, cols="int32")
    elif kind == "adjoint":
        levels = 3
        nx, ny, nz = _extents(rng, levels, 12, 48, True)
        c = dict(kind="adjoint", inner="fp32", nrhs=rng.choice([1, 1, 2, 4]), steps=0, cols="int32")
    else:
        levels = rng.choice([3, 4]) if kind == "vcycle" else rng.choice([1, 2])
        nx, ny, nz = _extents(rng, levels, 16, 250, kind != "smooth" and rng.random() < 0.7)
        nrhs = rng.choice([1, 1, 1, 4, 8]) if nx * ny * nz < 5_000_000 else 1
        inner = rng.choice(["fp64", "fp32", "fp32", "fp16", "bf16"] + (["fp16-mg", "bf16-mg"] if nrhs == 1 else []))
        c = dict(kind=kind, inner=inner, nrhs=nrhs, cols="int32")
    c.update(nx=nx, ny=ny, nz=nz, levels=levels, sweep=rng.choice(["forward", "forward", "backward", "symmetric"]))
    return c


# ---- inputs ----------------------------------------------------------------------------------------------
def _dims(case):
    return case["nx"], case["ny"], case["nz"]


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(case, g):
    nx, ny, nz = _dims(case)
    shape = (nx * ny * nz,) if case["nrhs"] == 1 else (case["nrhs"], nx * ny * nz)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)


def _theta(case, seed):
    """27 stencil entries: the benchmark's stencil, each off-diagonal entry a few percent off."""
    theta = torch.tensor(_beta_stencil(), dtype=torch.float64)
    g = torch.Generator()
    g.manual_seed(seed)
    noise = 1.0 + 0.05 * (torch.rand(27, generator=g, dtype=torch.float64) - 0.5)
    noise[13] = 1.02
    return theta * noise


def _vectors(case, seed):
    """The input vectors of a case, as run() gets them."""
    g = _gen(seed)
    u = _normal(case, g)
    if case["kind"] in ("vcycle", "smooth", "spmv"):
        vt = VEC.get(case["inner"], torch.float32)
        if case["kind"] == "smooth":
            return u.to(vt), _normal(case, g).to(vt)
        return (u.to(vt),)
    if case["kind"] == "adjoint":
        return u, _normal(case, g)
    return (u,)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "adjoint":
        theta = _theta(case, seed)
        solver = StencilSolver(_dims(case), levels=case["levels"], sweep=case["sweep"], tol=TOL)
        fwd, adj = solver.problems(theta)
        u, v = _vectors(case, seed)  # b = A u, dL/dx = A^T v
        rows = (lambda P, w: torch.stack([P.rhs_from_x(x) for x in w]) if w.dim() == 2 else P.rhs_from_x(w))
        return dict(case=case, solver=solver, b=rows(fwd, u).requires_grad_(), g=rows(adj, v),
                    theta=theta.cuda().requires_grad_())
    P = hpgmx.Problem(_dims(case), beta=BETA, levels=case["levels"], sweep=case["sweep"], cols=case["cols"])
    s = dict(case=case, P=P)
    v = _vectors(case, seed)
    if kind == "solve":
        u = v[0]
        s["b"] = P.rhs_from_x(u) if u.dim() == 1 else torch.stack([P.rhs_from_x(x) for x in u])
    else:
        s["r"] = v[0]
        s["z0"] = v[1] if kind == "smooth" else None
        s["z"] = torch.empty_like(v[0], dtype=torch.float32 if kind == "spmv" and "mg" in case["inner"] else None)
    return s


def run(s):
    case = s["case"]
    kind, batched, dt = case["kind"], case["nrhs"] > 1, DTYPE[case["inner"]]
    if kind == "adjoint":
        x = s["solver"](s["b"], s["theta"])
        gb, gt = torch.autograd.grad(x, (s["b"], s["theta"]), s["g"])
        return x.detach(), gb, gt
    P = s["P"]
    if kind == "solve":
        solve = P.solve_batched if batched else P.solve
        fixed = case["steps"] > 0
        x, _ = solve(s["b"], tol=1e-30 if fixed else TOL, restart=RESTART, precision=dt,
                     max_iters=case["steps"] if fixed else 2000, graph=P.N > 4096)
        return x
    sweep = SWEEP[case["sweep"]]
    if kind == "vcycle":
        (hpgmx.vcycle_batched if batched else hpgmx.vcycle)(P.h, dt, s["r"], s["z"])
    elif kind == "smooth":
        s["z"].copy_(s["z0"])
        (hpgmx.smooth_batched if batched else hpgmx.smooth)(P.h, 0, dt, sweep, s["r"], s["z"])
    else:
        (hpgmx.spmv_batched if batched else hpgmx.spmv)(P.h, 0, dt, s["r"], s["z"])
    return s["z"]


# ---- what a pass cannot do without ------------------------------------------------------------------------
def work(case):
    """Bytes: the stored matrix of every level the pass applies (values and column indices in the format the case
    asks for, once per application of the V-cycle and the operator), every input and output vector once, and in a
    solve the Krylov basis twice per inner step (an inner product needs a pass, the update that uses it another).
    Flops: two per stored entry and use, two per basis entry and pass."""
    nx, ny, nz = _dims(case)
    k, v = case["nrhs"], {"fp64": 8, "fp32": 4}.get(case["inner"], 2)
    w = {"fp64": 8, "fp16-mg": 2, "bf16-mg": 2}.get(case["inner"], 4)
    idx = 2 if case["cols"] == "offset16" else 4
    n = [(nx >> l) * (ny >> l) * (nz >> l) for l in range(case["levels"])]
    entry = 26 * (v + idx) + v
    kind, sweeps = case["kind"], 2 if case["sweep"] == "symmetric" else 1
    if kind == "spmv":
        return {"bytes": n[0] * (entry + 2 * k * w), "flops": n[0] * 54 * k}
    if kind == "smooth":
        return {"bytes": n[0] * (entry + 3 * k * w), "flops": n[0] * 54 * k * sweeps}
    cycle = sum(n) * entry
    cycle_flops = k * 54 * sweeps * (sum(2 * m for m in n[:-1]) + n[-1])
    if kind == "vcycle":
        return {"bytes": cycle + n[0] * 2 * k * w, "flops": cycle_flops}
    wk = max(w, 4)
    # a fixed count of steps, or about what 1e-11 takes from x = 0 on these grids
    steps = case["steps"] or int(20 * (n[0] / 4096) ** 0.32)
    solves = 2 if kind == "adjoint" else 1
    basis = sum(2 * (i % RESTART + 1) * n[0] * wk * k for i in range(steps))
    cycles = (steps + RESTART - 1) // RESTART
    outer = (cycles + 1) * n[0] * (26 * (8 + idx) + 8 + 3 * 8 * k)
    return {"bytes": solves * (steps * (cycle + 2 * n[0] * k * wk) + basis + outer),
            "flops": solves * (steps * (cycle_flops + 54 * k * n[0]) + basis / wk * 2)}


# ---- the same in FP64 with plain torch --------------------------------------------------------------------
def _beta_stencil(beta=BETA):
    c = []
    for t in range(27):
        di = t % 3 - 1
        c.append(26.0 if t == 13 else -1.0 - beta if di < 0 else -1.0 + beta if di > 0 else -1.0)
    return c


def _apply(c, x):
    """A x on a (nz, ny, nx) array."""
    nz, ny, nx = x.shape
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1, 1, 1))
    y = torch.zeros_like(x)
    for t, a in enumerate(c):
        di, dj, dk = t % 3, (t // 3) % 3, t // 9
        y += a * xp[dk:dk + nz, dj:dj + ny, di:di + nx]
    return y


def _relax(c, r, zp, colour):
    """One colour of Gauss-Seidel in place; zp is z with a border of zeros."""
    nz, ny, nx = r.shape
    pi, pj, pk = colour & 1, (colour >> 1) & 1, ((colour >> 2) & 1) ^ 1
    ni, nj, nk = len(range(pi, nx, 2)), len(range(pj, ny, 2)), len(range(pk, nz, 2))
    if ni * nj * nk == 0:
        return

    def at(di, dj, dk):
        i, j, k = 1 + pi + di, 1 + pj + dj, 1 + pk + dk
        return zp[k:k + 2 * nk - 1:2, j:j + 2 * nj - 1:2, i:i + 2 * ni - 1:2]

    acc = r[pk::2, pj::2, pi::2].clone()
    for t, a in enumerate(c):
        if t != 13:
            acc -= a * at(t % 3 - 1, (t // 3) % 3 - 1, t // 9 - 1)
    at(0, 0, 0).copy_(acc / c[13])


def _smooth(c, r, z, sweep):
    zp = torch.nn.functional.pad(z, (1, 1, 1, 1, 1, 1)).contiguous()
    order = {"forward": list(range(8)), "backward": list(range(7, -1, -1)),
             "symmetric": list(range(8)) + list(range(7, -1, -1))}[sweep]
    for colour in order:
        _relax(c, r, zp, colour)
    return zp[1:-1, 1:-1, 1:-1].contiguous()


def _vcycle(c, r, level, levels, sweep):
    z = _smooth(c, r, torch.zeros_like(r), sweep)
    if level == levels - 1:
        return z
    zc = _vcycle(c, (r - _apply(c, z))[::2, ::2, ::2].contiguous(), level + 1, levels, sweep)
    z[::2, ::2, ::2] += zc
    return _smooth(c, r, z, sweep)


def exact(case, seed):
    kind, (nx, ny, nz) = case["kind"], _dims(case)
    v = [x.to(torch.float64) for x in _vectors(case, seed)]
    if kind == "solve":
        return None if case["steps"] else v[0]  # b = A u: the solution is u
    if kind == "adjoint":
        u, lam = v  # b = A u and dL/dx = A^T lam
        xs = torch.nn.functional.pad(u.reshape(-1, nz, ny, nx), (1, 1, 1, 1, 1, 1))
        ls = lam.reshape(-1, nz, ny, nx)
        grad = torch.stack([-(ls * xs[:, t // 9:t // 9 + nz, (t // 3) % 3:(t // 3) % 3 + ny, t % 3:t % 3 + nx]).sum()
                            for t in range(27)])
        return u, lam, grad
    c = _beta_stencil()
    out = []
    for j in range(case["nrhs"]):
        w = [(x if case["nrhs"] == 1 else x[j]).reshape(nz, ny, nx) for x in v]
        if kind == "vcycle":
            y = _vcycle(c, w[0], 0, case["levels"], case["sweep"])
        elif kind == "smooth":
            y = _smooth(c, w[0], w[1], case["sweep"])
        else:
            y = _apply(c, w[0])
        out.append(y.reshape(-1))
    return out[0] if case["nrhs"] == 1 else torch.stack(out)
