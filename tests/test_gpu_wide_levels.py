"""Line kernels of the levels with more columns than the block forms take (a
wavefront or a pair of them per column tile), at every height class and its
edges: each launch shape against the oracle, the FP64 smoothers that meet in
the middle of the real rows against the smoothers that fold the prolongation.

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


# just above 16384 columns; tiles with remainders; two rows, three, each height
# class's first and last ragged height, odd and even, and the whole heights
GRIDS = [(136, 128, 2), (130, 127, 3), (130, 127, 5), (136, 128, 16), (130, 127, 17),
         (136, 128, 31), (130, 128, 33), (136, 128, 37), (130, 127, 64), (136, 128, 65),
         (130, 128, 70), (136, 127, 127), (136, 128, 128)]


@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid", GRIDS)
def test_smoother_shapes_match_oracle(grid, prec, bc_h):
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, orc, _ = problem(nx, ny, nz, seed=81, bc_h=bc_h)
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    u, f = W.uniform_pm1(81, 1, n), W.uniform_pm1(81, 2, n)
    if prec == 1:
        u, f = (a.astype(np.float32).astype(np.float64) for a in (u, f))
    bar = 1e-12 if prec == 0 else f32_line_bar(nz)
    fd, zd = ctx.to_device(f, dtype=dt), ctx.empty(dtype=dt)
    G.line_solve(ctx, 0, fd, zd)
    ref = orc.line_solve(f)
    assert max_rel(ctx.from_device(zd), ref, np.abs(ref).max()) < bar
    ref = orc.smooth(f, orc.smooth(f, u))
    # without a set shape, then the per-lane, two-wavefront and staged forms
    for shape in (None, (4, 0), (3, 0), (2, 0)):
        if shape is not None:
            G.gmg_set_launch(ctx, "smooth", 0, prec, *shape)
        ud = ctx.to_device(u, dtype=dt)
        G.line_smooth(ctx, 0, fd, ud, nsweeps=2)
        assert max_rel(ctx.from_device(ud), ref, np.abs(ref).max()) < 2 * bar


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("nz", [2, 5, 17, 33, 64, 70, 127, 128])
def test_folded_prolongation_equals_the_parts(nz, prec):
    """While the parts are timed, the prolongation and the smoother run as
    kernels of their own: bitwise the same V-cycle."""
    import paper_1402_3545_amd as G
    nx, ny = 136, 130
    ctx, orc, _ = problem(nx, ny, nz, nlevels=2, seed=83, prec_precond=prec)
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    fd = ctx.to_device(W.uniform_pm1(83, 1, n), dtype=dt)
    u = W.uniform_pm1(83, 2, n)
    outs = []
    for timed in (False, True):
        G.gmg_timing_enable(ctx, timed)
        ud = ctx.to_device(u, dtype=dt)
        G.gmg_vcycle(ctx, fd, ud)
        outs.append(ctx.from_device(ud))
    G.gmg_timing_enable(ctx, False)
    assert np.array_equal(outs[0], outs[1])
