"""Kernels at sizes where their dispatch changes: bitwise the values of another
launch shape, or within the oracle's bars (tests/test_gpu_kernels.py)."""

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


# 192, 224, 240 (whole and partial segments), 256 and 272 workgroups of 32 layers
@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid", [(256, 192, 32), (256, 224, 32), (192, 160, 64), (192, 160, 45),
                                  (256, 256, 32), (256, 272, 32)])
def test_prolongation_segments(grid, prec, bc_h):
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, _, _ = problem(nx, ny, nz, nlevels=2, seed=111, bc_h=bc_h)
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    uc = ctx.to_device(W.uniform_pm1(111, 1, n // 4), 1, dtype=dt)
    u0 = ctx.to_device(W.uniform_pm1(111, 2, n), dtype=dt)
    outs = []
    for rows in (4, 8):  # (8: always segments of 32 layers)
        G.gmg_set_launch(ctx, "prolongate", 1, prec, rows, 0)
        u = u0.clone()
        G.gmg_prolongate(ctx, 1, uc, u)
        outs.append(ctx.from_device(u))
    assert np.array_equal(*outs)


# FP32 smoothing of 128 layers: the last columns of the block form and the first
# of the other one
@pytest.mark.parametrize("bc_h", [0, 1])
@pytest.mark.parametrize("grid", [(128, 64, 128), (128, 65, 128), (128, 128, 128),
                                  (128, 65, 127)])
def test_fp32_smoothing_of_128_layers(grid, bc_h):
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, orc, _ = problem(nx, ny, nz, seed=113, bc_h=bc_h)
    n = nx * ny * nz
    f, u = (W.uniform_pm1(113, s, n).astype(np.float32).astype(np.float64) for s in (1, 2))
    fd, u0 = (ctx.to_device(v, dtype=torch.float32) for v in (f, u))
    ref = orc.smooth(f, orc.smooth(f, u))
    outs = []
    for shape in (None, (4, 0), (2, 0), (3, 0)):
        if shape:
            G.gmg_set_launch(ctx, "smooth", 0, G.GMG_F32, *shape)
        ud = u0.clone()
        G.line_smooth(ctx, 0, fd, ud, nsweeps=2)
        outs.append(ctx.from_device(ud))
    assert max_rel(outs[0], ref, np.abs(ref).max()) < 2 * f32_line_bar(nz)
    assert all(np.array_equal(o, outs[0]) for o in outs[1:])
