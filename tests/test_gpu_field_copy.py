"""An odd number of smoothing sweeps ends in the context's own buffer and is
copied back, large fields (from 32 MiB) in 16-byte words: bitwise the same as a single sweep at a time, and
no byte outside the field written, on sizes around a workgroup's share of the
copy (16 KiB) with its remainders."""

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid", [(2, 3, 2), (5, 7, 9), (16, 16, 8), (64, 16, 2), (64, 17, 4),
                                  (130, 127, 17), (514, 511, 33)])
def test_odd_sweeps(grid, prec):
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, _, _ = problem(nx, ny, nz, seed=91)
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    f = ctx.to_device(W.uniform_pm1(91, 1, n), dtype=dt)
    u0 = ctx.to_device(W.uniform_pm1(91, 2, n), dtype=dt)
    a, b = u0.clone(), u0.clone()
    # two sweeps leave the iterate in the caller's field, three in the buffer
    G.line_smooth(ctx, 0, f, a, nsweeps=2)
    G.line_smooth(ctx, 0, f, a, nsweeps=1)
    G.line_smooth(ctx, 0, f, b, nsweeps=3)
    # fields start at multiples of 16 bytes
    wide = torch.full((u0.numel() + 8,), 7.0, dtype=dt, device=u0.device)
    c = wide[4:-4]
    c.copy_(u0)
    G.line_smooth(ctx, 0, f, c, nsweeps=3)
    ref = ctx.from_device(a)
    assert np.array_equal(ref, ctx.from_device(b))
    assert np.array_equal(ref, ctx.from_device(c.clone()))
    assert bool((wide[:4] == 7.0).all()) and bool((wide[-4:] == 7.0).all())
