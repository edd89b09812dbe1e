"""Forms of the line kernels on levels above the block forms (more than 16384
columns; more than 32768 where an FP32 fold of at most 64 layers is meant): the
per-lane, staged and two-wavefront smoothers, the norm-computing smoother, the
folded prolongation and line-PCG's preconditioner step, each against another
form and against the oracle.

Bars: those of the line kernels (tests/test_gpu_kernels.py), of the folded
V-cycle (tests/test_gpu_prolong_smooth.py) and of the solver histories
(tests/test_gpu_solvers.py)."""

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


def _inputs(ctx, seed, n, prec):
    dt = torch.float64 if prec == 0 else torch.float32
    f, u = W.uniform_pm1(seed, 1, n), W.uniform_pm1(seed, 2, n)
    if prec == 1:
        f, u = (a.astype(np.float32).astype(np.float64) for a in (f, u))
    return f, u, ctx.to_device(f, dtype=dt), ctx.to_device(u, dtype=dt)


# 33280 columns, whole tiles of 64 columns by 2 rows: the two-wavefront form
# fits (the last tile row of the four-row forms is half empty)
WX, WY = 256, 130


@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nz", [32, 64, 128])
def test_two_wavefront_smoother(nz, prec, bc_h):
    """Per-lane, staged and two-wavefront sweeps: bitwise the same iterate, in
    any tile order, and the oracle's."""
    import paper_1402_3545_amd as G
    ctx, orc, _ = problem(WX, WY, nz, seed=101, bc_h=bc_h)
    f, u, fd, u0 = _inputs(ctx, 101, WX * WY * nz, prec)
    outs = []
    for shape in (None, (4, 0), (2, 0), (3, 0), (3, 2)):
        if shape:
            G.gmg_set_launch(ctx, "smooth", 0, prec, *shape)
        ud = u0.clone()
        G.line_smooth(ctx, 0, fd, ud, nsweeps=2)
        outs.append(ctx.from_device(ud))
    assert all(np.array_equal(o, outs[0]) for o in outs[1:])
    ref = orc.smooth(f, orc.smooth(f, u))
    bar = 1e-12 if prec == 0 else f32_line_bar(nz)
    assert max_rel(outs[0], ref, np.abs(ref).max()) < 2 * bar


@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nz", [32, 64, 128])
def test_two_wavefront_fold(nz, prec, bc_h):
    """The post-smoother with the prolongation folded in, by one and by two
    wavefronts a column, against the two kernels and the oracle's cycle."""
    import paper_1402_3545_amd as G
    ctx, orc, _ = problem(WX, WY, nz, nlevels=2, seed=103, bc_h=bc_h, prec_precond=prec)
    f, u, fd, u0 = _inputs(ctx, 103, WX * WY * nz, prec)
    outs = []
    for shape in (None, (4, 0), (2, 0), (3, 0), (3, 2)):
        if shape:
            G.gmg_set_launch(ctx, "prolong_smooth", 0, prec, *shape)
        ud = u0.clone()
        G.gmg_vcycle(ctx, fd, ud)
        outs.append(ctx.from_device(ud))
    assert all(np.array_equal(o, outs[0]) for o in outs[1:])
    ref = orc.vcycle(f, u)
    assert max_rel(outs[0], ref, np.abs(ref).max()) < (1e-11 if prec == 0 else 1e-4)


# the norm-computing smoother in each form, at whole heights (two wavefronts)
# and at ragged ones, where the FP64 halves meet in the middle of the real rows
@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("grid", [(WX, WY, 32), (WX, WY, 128), (136, 130, 2), (136, 130, 5),
                                  (136, 130, 37), (136, 130, 70), (136, 130, 127)])
def test_multigrid_solve_by_each_smoother(grid, bc_h):
    """Residual history, stopping cycle and solution of the FP64 multigrid
    solve, whose stopping test is the norm taken by its smoother."""
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, orc, _ = problem(nx, ny, nz, nlevels=2, seed=105, bc_h=bc_h)
    f = W.rhs(105, 0, nx, ny, nz)
    fd = ctx.to_device(f)
    _, _, full, _ = orc.mg_solve(f, rtol=1e-300, maxit=6)
    rtol = float(np.sqrt(full[3] * full[4]))   # between the third and fourth cycle
    u_ref, it_ref, hist_ref, st_ref = orc.mg_solve(f, rtol=rtol, maxit=50)
    assert st_ref == 0 and it_ref == 4
    hists = []
    for shape in (None, (4, 0), (2, 0), (3, 0)):
        if shape:
            G.gmg_set_launch(ctx, "smooth", 0, G.GMG_F64, *shape)
        ud = ctx.empty()
        it, rel, hist, st = G.gmg_solve(ctx, fd, ud, rtol=rtol, maxit=50)
        assert st == 0 and it == it_ref, shape
        np.testing.assert_allclose(hist, hist_ref, rtol=1e-9, atol=0)
        assert max_rel(ctx.from_device(ud), u_ref, np.abs(u_ref).max()) < 1e-9
        hists.append(hist)
    # the forms differ in the order of their partial sums only
    assert all(np.allclose(h, hists[0], rtol=1e-12, atol=0) for h in hists)


# ragged and whole heights of each class; fields above the FP32 fold's limit for
# at most 64 layers, and above that for more
FOLDS = [(WX, WY, 2), (WX, WY, 5), (WX, WY, 17), (WX, WY, 37), (WX, WY, 63),
         (136, 130, 65), (136, 130, 70), (136, 130, 127), (136, 130, 128)]


@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid", FOLDS)
def test_staged_fold(grid, prec, bc_h):
    """The staged smoother with the prolongation folded in, asked for by its
    launch shape: bitwise the cycle of the two kernels, and the oracle's."""
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, orc, _ = problem(nx, ny, nz, nlevels=2, seed=107, bc_h=bc_h, prec_precond=prec)
    f, u, fd, u0 = _inputs(ctx, 107, nx * ny * nz, prec)
    outs = []
    for shape in ((4, 0), (2, 0), (2, 2), (3, 0)):
        G.gmg_set_launch(ctx, "prolong_smooth", 0, prec, *shape)
        ud = u0.clone()
        G.gmg_vcycle(ctx, fd, ud)
        outs.append(ctx.from_device(ud))
    assert all(np.array_equal(o, outs[0]) for o in outs[1:])
    ref = orc.vcycle(f, u)
    assert max_rel(outs[0], ref, np.abs(ref).max()) < (1e-11 if prec == 0 else 1e-4)


# above 8192 columns the preconditioner step takes two lanes a column
@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("grid", [(100, 90, 33), (136, 130, 2), (136, 130, 5), (136, 130, 37),
                                  (136, 130, 70), (136, 130, 127)])
def test_pcg_at_ragged_heights(grid, bc_h):
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, orc, _ = problem(nx, ny, nz, seed=109, bc_h=bc_h)
    f = W.rhs(109, 0, nx, ny, nz)
    ud = ctx.empty()
    it, rel, hist, st = G.pcg_solve(ctx, ctx.to_device(f), ud, rtol=1e-8, maxit=500)
    u_ref, it_ref, hist_ref, _, st_ref = orc.pcg_solve(f, rtol=1e-8, maxit=500)
    assert st == st_ref == 0 and it == it_ref
    np.testing.assert_allclose(hist, hist_ref, rtol=1e-6, atol=1e-14)
    assert max_rel(ctx.from_device(ud), u_ref, np.abs(u_ref).max()) < 1e-9


# the line solve keeps two lanes a column above 8192 columns and 64 layers, and
# above 16384 columns throughout
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid", [(100, 90, 65), (100, 90, 70), (100, 90, 127), (100, 90, 128),
                                  (136, 130, 37), (WX, WY, 64)])
def test_tile_orders_of_the_line_kernels(grid, prec):
    """Line solve and smoother in every tile order: bitwise the same values, and
    the oracle's."""
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, orc, _ = problem(nx, ny, nz, seed=115)
    f, u, fd, u0 = _inputs(ctx, 115, nx * ny * nz, prec)
    outs = []
    for group in (0, 1, 2, 8):
        G.gmg_set_launch(ctx, "line_solve", 0, prec, 4, group)
        zd = ctx.empty(dtype=fd.dtype)
        G.line_solve(ctx, 0, fd, zd)
        res = [ctx.from_device(zd)]
        for rows in (4, 2):
            G.gmg_set_launch(ctx, "smooth", 0, prec, rows, group)
            ud = u0.clone()
            G.line_smooth(ctx, 0, fd, ud, nsweeps=2)
            res.append(ctx.from_device(ud))
        outs.append(res)
    for res in outs:
        assert np.array_equal(res[0], outs[0][0])
        assert np.array_equal(res[1], outs[0][1]) and np.array_equal(res[2], outs[0][1])
    bar = 1e-12 if prec == 0 else f32_line_bar(nz)
    ref = orc.line_solve(f)
    assert max_rel(outs[0][0], ref, np.abs(ref).max()) < bar
    ref = orc.smooth(f, orc.smooth(f, u))
    assert max_rel(outs[0][1], ref, np.abs(ref).max()) < 2 * bar


@pytest.mark.parametrize("nz", [37, 64])
def test_tile_orders_of_the_cg_step(nz):
    """Line-PCG with its preconditioner step in every tile order: the same
    iteration count, the solutions equal to the rounding of its dot products
    (which group other columns)."""
    import paper_1402_3545_amd as G
    nx, ny = 136, 130
    ctx, orc, _ = problem(nx, ny, nz, seed=117)
    f = W.rhs(117, 0, nx, ny, nz)
    fd = ctx.to_device(f)
    u_ref, it_ref, hist_ref, _, st_ref = orc.pcg_solve(f, rtol=1e-8, maxit=500)
    for group in (0, 1, 2, 8):
        G.gmg_set_launch(ctx, "cg_tridiag", 0, G.GMG_F64, 4, group)
        ud = ctx.empty()
        it, rel, hist, st = G.pcg_solve(ctx, fd, ud, rtol=1e-8, maxit=500)
        assert st == st_ref == 0 and it == it_ref
        np.testing.assert_allclose(hist, hist_ref, rtol=1e-6, atol=1e-14)
        assert max_rel(ctx.from_device(ud), u_ref, np.abs(u_ref).max()) < 1e-9
