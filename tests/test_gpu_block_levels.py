"""Line kernels of the levels with few columns (a workgroup per 8, 16 or 32
columns) at the sizes where their dispatch and their tiles change, against the
oracle, and the fused residual + restriction + line solve against the kernels
it stands for.

Bars: those of the line kernels (tests/test_gpu_kernels.py)."""

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import f32_line_bar, max_rel, problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")


# columns: below a workgroup, a remainder of 8, the last grids with 8 and 16
# columns a workgroup and the first with more, remainders of 16 and 32, the
# largest line solve and smoother; layers: every height class and its edges
GRIDS = [(2, 3, 2), (5, 7, 9), (64, 32, 128), (43, 48, 33), (64, 64, 64), (65, 64, 16),
         (128, 64, 17), (127, 129, 5), (128, 128, 8)]


@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid", GRIDS)
def test_solve_and_smooth_match_oracle(grid, prec, bc_h):
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, orc, _ = problem(nx, ny, nz, seed=71, bc_h=bc_h)
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    u, f = W.uniform_pm1(71, 1, n), W.uniform_pm1(71, 2, n)
    if prec == 1:
        u, f = (a.astype(np.float32).astype(np.float64) for a in (u, f))
    ud, fd, zd = ctx.to_device(u, dtype=dt), ctx.to_device(f, dtype=dt), ctx.empty(dtype=dt)
    bar = 1e-12 if prec == 0 else f32_line_bar(nz)
    G.line_solve(ctx, 0, fd, zd)
    ref = orc.line_solve(f)
    assert max_rel(ctx.from_device(zd), ref, np.abs(ref).max()) < bar
    G.line_smooth(ctx, 0, fd, ud, nsweeps=2)
    ref = orc.smooth(f, orc.smooth(f, u))
    assert max_rel(ctx.from_device(ud), ref, np.abs(ref).max()) < 2 * bar


# a coarse level of one column, of a remainder, at the largest fused size and
# beyond it; ragged and whole column heights
@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid,L", [((2, 2, 9), 2), ((40, 24, 37), 3), ((8, 8, 128), 4),
                                    ((96, 72, 3), 2), ((256, 256, 16), 3), ((258, 256, 5), 2)])
def test_fused_levels_equal_their_parts(grid, L, prec, bc_h):
    """While the parts are timed, the restriction, the line solve, the
    prolongation and the smoother run as kernels of their own: bitwise the same
    V-cycle."""
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, orc, _ = problem(nx, ny, nz, nlevels=L, seed=73, bc_h=bc_h, prec_precond=prec)
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    fd = ctx.to_device(W.uniform_pm1(73, 1, n), dtype=dt)
    u = W.uniform_pm1(73, 2, n)
    outs = []
    for timed in (False, True):
        G.gmg_timing_enable(ctx, timed)
        ud = ctx.to_device(u, dtype=dt)
        G.gmg_vcycle(ctx, fd, ud)
        outs.append(ctx.from_device(ud))
    kinds = {k[0] for k in G.gmg_timing_table(ctx)}
    G.gmg_timing_enable(ctx, False)
    assert {"residual_restrict", "line_solve", "prolongate", "smooth"} <= kinds
    assert np.array_equal(outs[0], outs[1])


def test_small_pcg_matches_oracle():
    """The preconditioner step of line-PCG on a grid of few columns."""
    import paper_1402_3545_amd as G
    nx, ny, nz = 44, 37, 50
    ctx, orc, _ = problem(nx, ny, nz, seed=75)
    f = W.rhs(75, 0, nx, ny, nz)
    ud = ctx.empty()
    it, rel, hist, st = G.pcg_solve(ctx, ctx.to_device(f), ud, rtol=1e-8, maxit=500)
    u_ref, it_ref, hist_ref, _, st_ref = orc.pcg_solve(f, rtol=1e-8, maxit=500)
    assert st == st_ref == 0 and it == it_ref
    np.testing.assert_allclose(hist, hist_ref, rtol=1e-6, atol=1e-14)
    assert max_rel(ctx.from_device(ud), u_ref, np.abs(u_ref).max()) < 1e-9


@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("nz", [9, 37, 64, 128])
def test_batched_levels_equal_single_solves(nz, bc_h):
    """Grouped launches whose levels are above and below the line of the block
    forms (here 3 x 64^2 and 64 x 192 columns, then a quarter of that): the same
    cycles as single-instance contexts."""
    import paper_1402_3545_amd as G
    kws = [dict(nx=nx, ny=ny, nz=nz, nlevels=L, kv=1e3, bc_h=bc_h,
                kh=W.kh_uniform(80 + q, nx, ny), zfaces=W.quadratic_faces(nz))
           for q, (nx, ny, L) in enumerate([(64, 64, 3), (64, 192, 2), (64, 64, 1), (40, 24, 3)])]
    b = G.gmg_batch_setup([dict(prec_precond=1, **kw) for kw in kws], nrhs=2)
    fh, fs, us = [], [], []
    for q, kw in enumerate(kws):
        for r in range(2):
            fh.append(W.rhs(80 + q, r, kw["nx"], kw["ny"], nz))
            fs.append(b.to_device(fh[-1], q))
            us.append(b.empty(q))
    it, rel, st = G.gmg_batch_solve(b, fs, us, rtol=1e-8, maxit=60)
    assert st == 0
    for p, u in enumerate(us):
        ctx = G.GmgContext(prec_precond=G.GMG_F32, **kws[p // 2])
        ud = ctx.empty()
        it1, _, _, st1 = G.gmg_solve(ctx, ctx.to_device(fh[p]), ud, rtol=1e-8, maxit=60)
        u1, ub = ctx.from_device(ud), b.from_device(u, p // 2)
        assert st1 == 0 and it1 == it[p]
        assert np.abs(u1 - ub).max() <= 1e-12 * np.abs(u1).max()
