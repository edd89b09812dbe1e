"""The calls whose speed is measured: what programs built on this library have it do.

A program keeps a context (or a batched context) and device fields, and calls
single operations, V-cycles or whole solves on them.  The cases run from one
smoothing call on a small grid, which is all latency, to the 2048^2 x 128 solve;
grids whose sizes are no multiple of a wavefront, both boundary types, both
precisions and every solver are among them.

`exact` computes the same results in float64 with plain torch operations.
"""

import math
import random

import numpy as np
import torch

import paper_1402_3545_amd as G

RHO = 2.0 / 3.0

# kind: what one pass calls.  model: "graded" is the periodic operator with
# K_T ~ U[0.5, 2] and quadratically graded layers, "lognormal" the same with
# K_T = exp(N(0, 1/4)), "flatbox" the paper's model problem (Dirichlet side
# walls, Neumann ends, nu_CFL = 8.4).  stored: apply the launch shapes stored
# for the grid, as the benchmark does; otherwise the context is used as set up.
_DEFAULTS = dict(model="graded", kv=1e4, levels=1, prec=0, rtol=1e-8, stored=False)


def _case(name, kind, nx, ny, nz, **kw):
    c = dict(_DEFAULTS, kind=kind, nx=nx, ny=ny, nz=nz)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # two sweeps of the smoother on a small ragged grid inside a caller's own iteration
        _case("smooth-f32-40x24x37", "smooth", 40, 24, 37, kv=1e3, prec=1),
        # the steps of Algorithm 1 called one by one, by a program with its own cycle
        _case("twogrid-f64-512x384x64", "twogrid", 512, 384, 64, levels=2),
        # one FP32 cycle as a preconditioner in a caller's own Krylov loop, ragged sizes
        _case("vcycle-f32-200x120x50", "vcycle", 200, 120, 50, levels=3, prec=1),
        # the small cache-resident workload, solved to five digits
        _case("mg-64x64x64", "mg", 64, 64, 64, levels=4, kv=1e3, rtol=1e-5),
        # line-PCG on the smallest grid of the paper's single-GPU table
        _case("pcg-flatbox-128x128x128", "pcg", 128, 128, 128, model="flatbox", rtol=1e-5),
        # the CFL study's deepest hierarchy, down to one column
        _case("mg-flatbox-512x512x128", "mg", 512, 512, 128, levels=10, model="flatbox",
              rtol=1e-5, stored=True),
        # total solution time from host memory
        _case("host-256x256x64", "host", 256, 256, 64, levels=4),
        # several instances with several right-hand sides each
        _case("batch-8x4", "batch", 512, 512, 128, ninst=8, nrhs=4, prec=1),
        # one GPU's share of the benchmark, by three of its solvers
        _case("mg-1024x1024x128", "mg", 1024, 1024, 128, levels=6, stored=True),
        _case("fcg-1024x1024x128", "fcg", 1024, 1024, 128, levels=6, prec=1, stored=True),
        _case("pcg-1024x1024x128", "pcg", 1024, 1024, 128, levels=6, stored=True),
        # the largest grid, FP32 cycles in FP64 refinement
        _case("refine-2048x2048x128", "mg", 2048, 2048, 128, levels=7, prec=1,
              model="lognormal", kv=1e5, stored=True),
    ]


def draw(rng):
    kind = rng.choice(["smooth", "twogrid", "vcycle", "mg", "mg", "pcg", "fcg", "host", "batch"])
    prec = rng.randint(0, 1)
    if kind == "batch":
        n = rng.choice([128, 192, 256, 320, 384, 512])
        return _case(None, kind, n, n, rng.choice([32, 45, 64, 100, 128]),
                     ninst=rng.randint(2, 8), nrhs=rng.randint(1, 4), prec=1)

    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    nz = rng.choice([32, 64, 128, spread(9, 128), spread(9, 128)])
    nx = spread(24, 800)
    ny = min(800, max(24, int(nx * rng.uniform(0.6, 1.7))))
    # hierarchies down to 12 to 24 columns a side; one level where none is used
    levels = 1 if kind in ("smooth", "pcg") else max(2, int(math.log2(min(nx, ny) / 12)) + 1)
    unit = 1 << (levels - 1)
    nx, ny = nx // unit * unit, ny // unit * unit
    if kind in ("host", "fcg"):
        prec = 1 if kind == "fcg" else 0
    model = rng.choice(["graded", "graded", "flatbox"])
    if model == "flatbox":
        ny = nx  # the model problem's box is square, with one CFL number
    return _case(None, kind, nx, ny, nz, model=model, levels=levels, prec=prec,
                 kv=rng.choice([1e3, 1e4]), rtol=1e-5 if model == "flatbox" else 1e-8)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _operator(case, seed):
    """The keyword arguments that define the operator, drawn from the seed."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    rng = np.random.default_rng(seed)
    if case["model"] == "flatbox":
        k = (0.5 * 8.4 / nx) ** 2
        return dict(kv=k, kh=np.full(nx * ny, k), zfaces=10.0 / 6371.0 * np.arange(nz + 1) / nz,
                    bc_h=1, bc_v=1)
    if case["model"] == "lognormal":
        kh = np.exp(0.5 * rng.standard_normal(nx * ny))
    else:
        kh = rng.uniform(0.5, 2.0, nx * ny)
    return dict(kv=case["kv"], kh=kh, zfaces=(np.arange(nz + 1) / nz) ** 2, bc_h=0, bc_v=0)


def _values(case, seed, stream, level=0, f32=False):
    """Uniform values in [-1, 1] for the cells of a level, (ny, nz, nx)."""
    g = torch.Generator(device=_device())
    g.manual_seed(1000003 * (int(seed) + 1) + stream)
    shape = (case["ny"] >> level, case["nz"], case["nx"] >> level)
    v = torch.rand(shape, generator=g, device=_device(), dtype=torch.float64)
    v = v.mul_(2.0).sub_(1.0)
    return v.float() if f32 else v


def _instances(case, seed):
    """The batch's instances as cases of their own: square grids up to the case's,
    coarsened while the size stays at least 32 and even."""
    rng = random.Random(case["ninst"] * 64 + case["nrhs"])
    out = []
    for q in range(case["ninst"]):
        n = max(32, case["nx"] >> rng.randint(0, 2))
        levels = 1
        while n % (1 << levels) == 0 and n >> levels >= 32:
            levels += 1
        out.append(dict(case, nx=n, ny=n, nz=max(16, case["nz"] >> rng.randint(0, 1)),
                        levels=levels))
    return out


def _field(values, ldx, dtype=None):
    ny, nz, nx = values.shape
    t = torch.zeros((ny, nz, ldx), dtype=dtype or values.dtype, device=values.device)
    t[:, :, :nx] = values
    return t.view(-1)


def _cells(t, ctx, level=0):
    nx, ny, nz = ctx.shape(level)
    return t.view(ny, nz, -1)[:, :, :nx]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        inst = _instances(case, seed)
        b = G.gmg_batch_setup([dict(nx=c["nx"], ny=c["ny"], nz=c["nz"], nlevels=c["levels"],
                                    prec_precond=1, **_operator(c, seed + q))
                               for q, c in enumerate(inst)], nrhs=case["nrhs"])
        fs, us = [], []
        for q, c in enumerate(inst):
            for r in range(case["nrhs"]):
                fs.append(_field(_values(c, seed, 16 + q * case["nrhs"] + r), b.layout(q)[0]))
                us.append(b.empty(q))
        return dict(case=case, batch=b, f=fs, u=us, inst=inst)
    ctx = G.gmg_setup(nx=case["nx"], ny=case["ny"], nz=case["nz"], nlevels=case["levels"],
                      prec_precond=case["prec"], **_operator(case, seed))
    if case["stored"]:
        G.tuned(ctx)
    s = dict(case=case, ctx=ctx)
    if kind == "host":
        s["f"] = _values(case, seed, 1).permute(0, 2, 1).contiguous().cpu().numpy().reshape(-1)
        s["u"] = np.zeros_like(s["f"])
        return s
    solver = kind in ("mg", "pcg", "fcg")
    f32 = case["prec"] == 1 and not solver
    ldx = ctx.layout()[0]
    s["f"] = _field(_values(case, seed, 1, f32=f32), ldx)
    if solver:
        s["u"] = ctx.empty()
    else:
        s["u"] = _field(_values(case, seed, 2, f32=f32), ldx)
    if kind == "twogrid":
        dt = s["f"].dtype
        s["r"], s["fc"], s["uc"] = (ctx.empty(dtype=dt), ctx.empty(1, dtype=dt),
                                    ctx.empty(1, dtype=dt))
    return s


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def run(s):
    case = s["case"]
    kind, f, u = case["kind"], s["f"], s["u"]
    if kind == "batch":
        for t in u:
            t.zero_()
        it, _, _ = G.gmg_batch_solve(s["batch"], f, u, rtol=case["rtol"], maxit=100)
        return dict(iterations=it, u=[
            t.view(c["ny"], c["nz"], -1)[:, :, :c["nx"]]
            for t, c in zip(u, [c for c in s["inst"] for _ in range(case["nrhs"])])])
    ctx = s["ctx"]
    if kind == "smooth":
        G.line_smooth(ctx, 0, f, u, nsweeps=2)
        return dict(u=_cells(u, ctx))
    if kind == "vcycle":
        G.gmg_vcycle(ctx, f, u)
        return dict(u=_cells(u, ctx))
    if kind == "twogrid":
        G.line_smooth(ctx, 0, f, u)
        G.gmg_residual(ctx, 0, f, u, s["r"])
        G.gmg_restrict_smooth(ctx, 1, s["r"], s["fc"], s["uc"])
        G.gmg_prolongate(ctx, 1, s["uc"], u)
        G.line_smooth(ctx, 0, f, u)
        return dict(u=_cells(u, ctx), r=_cells(s["r"], ctx), fc=_cells(s["fc"], ctx, 1),
                    uc=_cells(s["uc"], ctx, 1))
    if kind == "host":
        u.fill(0.0)
        it, _, _, _ = G.gmg_solve_host(ctx, f, u, rtol=case["rtol"])
        return dict(iterations=it, u=u)
    u.zero_()
    if kind == "mg":
        it = G.gmg_solve(ctx, f, u, rtol=case["rtol"], maxit=100)[0]
    else:
        it = G.pcg_solve(ctx, f, u, rtol=case["rtol"], maxit=1000,
                         precond=1 if kind == "fcg" else 0)[0]
    return dict(iterations=it, u=_cells(u, ctx))


# ---------------------------------------------------------------------------
# Work: each step of the algorithms reads its inputs and writes its outputs once
# ---------------------------------------------------------------------------
def work(case):
    if case["kind"] == "batch":
        parts = [work(dict(c, kind="mg")) for c in _instances(case, 0)]
        return {k: case["nrhs"] * sum(p[k] for p in parts) for k in ("bytes", "flops")}
    n = case["nx"] * case["ny"] * case["nz"]
    w = 4 if case["prec"] else 8
    tail = 4.0 / 3.0 if case["levels"] > 1 else 1.0
    # smooth, residual + restriction, prolongation + smooth: 3 + 2.25 + 3.25 words a cell
    cycle = 8.5 * tail * w * n
    digits = math.log(1.0 / case["rtol"])
    cycles = max(1, round(digits / math.log(2.64)))
    if case["kind"] == "smooth":
        return dict(bytes=2 * 3 * w * n, flops=2 * 40 * n)
    if case["kind"] == "vcycle":
        return dict(bytes=cycle, flops=90 * tail * n)
    if case["kind"] == "twogrid":
        # smooth 3, residual 3, restriction + coarse solve 1.5, prolongation 2.25, smooth 3
        return dict(bytes=12.75 * w * n, flops=110 * n)
    if case["kind"] == "mg":
        # refinement adds u, f, u' in FP64 and e, r in FP32 to each FP32 cycle
        per = cycle + (32 * n if case["prec"] else 0)
        return dict(bytes=cycles * per, flops=cycles * 110 * tail * n)
    if case["kind"] == "host":
        return dict(bytes=cycles * cycle + 24 * n, flops=cycles * 90 * tail * n)
    if case["kind"] == "fcg":
        its = max(1, cycles // 2)
        return dict(bytes=its * (cycle + 96 * n), flops=its * 130 * tail * n)
    # line-PCG: direction step 6.5, preconditioner step 4 words a cell and iteration
    its = max(1, round(4.4 * digits))
    return dict(bytes=its * 10.5 * 8 * n, flops=its * 60 * n)


# ---------------------------------------------------------------------------
# The same results in float64 with plain torch operations
# ---------------------------------------------------------------------------
class _Level:
    """One level of the hierarchy; fields are (nz, ny, nx)."""

    def __init__(self, K, op, nz):
        ny, nx = K.shape
        hx, hy = 1.0 / nx, 1.0 / ny
        z = torch.from_numpy(np.asarray(op["zfaces"], dtype=np.float64)).to(K)
        dz = z[1:] - z[:-1]
        mid = 0.5 * (z[1:] + z[:-1])
        t = torch.zeros(nz + 1).to(K)
        t[1:nz] = op["kv"] / (mid[1:] - mid[:-1])
        if op["bc_v"] == 0:
            t[0], t[nz] = 2.0 * op["kv"] / dz[0], 2.0 * op["kv"] / dz[-1]
        self.walls, self.dz, self.off = op["bc_h"] == 1, dz, -hx * hy * t[1:nz]

        def mean(dim):
            o = torch.roll(K, -1, dim)
            return 2.0 * K * o / (K + o)

        self.ce, self.cn = hy / hx * mean(1), hx / hy * mean(0)
        S = torch.zeros_like(K)
        if self.walls:
            self.ce[:, -1] = 0.0
            self.cn[-1, :] = 0.0
            for edge, ratio in ((np.s_[:, 0], hy / hx), (np.s_[:, -1], hy / hx),
                                (np.s_[0, :], hx / hy), (np.s_[-1, :], hx / hy)):
                S[edge] += ratio * 2.0 * K[edge]
        if nx == 1:
            self.ce.zero_()
        if ny == 1:
            self.cn.zero_()
        self.cw, self.cs = torch.roll(self.ce, 1, 1), torch.roll(self.cn, 1, 0)
        S += self.ce + self.cw + self.cn + self.cs
        self.diag = (hx * hy * (dz + t[:-1] + t[1:])).view(-1, 1, 1) + dz.view(-1, 1, 1) * S
        # the elimination of every column, once
        self.inv, self.cp = torch.empty_like(self.diag), torch.empty_like(self.diag)
        for k in range(nz):
            p = self.diag[k] if k == 0 else self.diag[k] - self.off[k - 1] * self.cp[k - 1]
            self.inv[k] = 1.0 / p
            if k + 1 < nz:
                self.cp[k] = self.off[k] * self.inv[k]

    def residual(self, f, u):
        h = self.ce * torch.roll(u, -1, 2)
        h += self.cw * torch.roll(u, 1, 2)
        h += self.cn * torch.roll(u, -1, 1)
        h += self.cs * torch.roll(u, 1, 1)
        r = f - self.diag * u + self.dz.view(-1, 1, 1) * h
        off = self.off.view(-1, 1, 1)
        r[1:] -= off * u[:-1]
        r[:-1] -= off * u[1:]
        return r

    def solve(self, r):
        x = torch.empty_like(r)
        nz = r.shape[0]
        x[0] = r[0] * self.inv[0]
        for k in range(1, nz):
            x[k] = (r[k] - self.off[k - 1] * x[k - 1]) * self.inv[k]
        for k in range(nz - 2, -1, -1):
            x[k] -= self.cp[k] * x[k + 1]
        return x

    def smooth(self, f, u):
        return u + RHO * self.solve(self.residual(f, u))


def _restrict(r):
    return r[:, 0::2, 0::2] + r[:, 0::2, 1::2] + r[:, 1::2, 0::2] + r[:, 1::2, 1::2]


def _prolong(c, walls):
    for dim in (1, 2):
        lo, hi = torch.roll(c, 1, dim), torch.roll(c, -1, dim)
        if walls:
            n = c.shape[dim]
            lo.narrow(dim, 0, 1).copy_(-c.narrow(dim, 0, 1))
            hi.narrow(dim, n - 1, 1).copy_(-c.narrow(dim, n - 1, 1))
        pair = torch.stack((0.75 * c + 0.25 * lo, 0.75 * c + 0.25 * hi), dim + 1)
        c = pair.flatten(dim, dim + 1)
    return c


class _Exact:
    def __init__(self, case, op):
        K = torch.from_numpy(np.asarray(op["kh"])).to(_device()).view(case["ny"], case["nx"])
        self.lev = []
        for _ in range(case["levels"]):
            self.lev.append(_Level(K, op, case["nz"]))
            K = 0.25 * _restrict(K.unsqueeze(0))[0] if len(self.lev) < case["levels"] else K

    def cycle(self, f, u, d=0):
        """One V(1,1) cycle on level d; u None: from a zero guess."""
        A = self.lev[d]
        u = RHO * A.solve(f) if u is None else A.smooth(f, u)
        if d == len(self.lev) - 1:
            return A.smooth(f, u)
        u = u + _prolong(self.cycle(_restrict(A.residual(f, u)), None, d + 1), A.walls)
        return A.smooth(f, u)

    def mg(self, f, rtol):
        A, u, r0 = self.lev[0], torch.zeros_like(f), f.norm()
        for _ in range(100):
            u = self.cycle(f, u)
            if A.residual(f, u).norm() < rtol * r0:
                break
        return u

    def cg(self, f, rtol, precond):
        """Conjugate gradients; with one direction kept, the flexible form."""
        A, u, r, r0 = self.lev[0], torch.zeros_like(f), f.clone(), f.norm()
        p = q = s = None
        for _ in range(1000):
            z = precond(r)
            p = z if p is None else z - (z * q).sum() / s * p
            q = -A.residual(torch.zeros_like(p), p)
            s = (p * q).sum()
            alpha = (p * r).sum() / s
            u += alpha * p
            r -= alpha * q
            if r.norm() < rtol * r0:
                break
        return u


def exact(case, seed):
    kind = case["kind"]

    def zyx(v):
        return v.double().permute(1, 0, 2).contiguous()

    def out(v):
        return v.permute(1, 0, 2)

    if kind == "batch":
        us = []
        for q, c in enumerate(_instances(case, seed)):
            E = _Exact(c, _operator(c, seed + q))
            us += [out(E.mg(zyx(_values(c, seed, 16 + q * case["nrhs"] + r)), c["rtol"]))
                   for r in range(case["nrhs"])]
        return dict(iterations=None, u=us)
    E = _Exact(case, _operator(case, seed))
    f32 = case["prec"] == 1 and kind in ("smooth", "vcycle", "twogrid")
    f = zyx(_values(case, seed, 1, f32=f32))
    A = E.lev[0]
    if kind in ("smooth", "vcycle", "twogrid"):
        u = zyx(_values(case, seed, 2, f32=f32))
        if kind == "smooth":
            return dict(u=out(A.smooth(f, A.smooth(f, u))))
        if kind == "vcycle":
            return dict(u=out(E.cycle(f, u)))
        u = A.smooth(f, u)
        r = A.residual(f, u)
        fc = _restrict(r)
        uc = RHO * E.lev[1].solve(fc)
        u = A.smooth(f, u + _prolong(uc, A.walls))
        return dict(u=out(u), r=out(r), fc=out(fc), uc=out(uc))
    if kind == "host":
        return dict(iterations=None,
                    u=E.mg(f, case["rtol"]).permute(1, 2, 0).contiguous().cpu().numpy().reshape(-1))
    if kind == "mg":
        u = E.mg(f, case["rtol"])
    elif kind == "pcg":
        u = E.cg(f, case["rtol"], A.solve)
    else:
        u = E.cg(f, case["rtol"], lambda r: E.cycle(r, None))
    return dict(iterations=None, u=out(u))
