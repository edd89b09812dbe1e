"""The V-cycle's fused launches (restriction with the coarse line solve,
prolongation with the post-smoother): what is timed is what runs."""

import numpy as np
import pytest

import workloads as W
from tests.gpu_util import max_rel, problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True, scope="module")
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")


def _launched(G, ctx, fn):
    """{kind: launches} of fn as an untimed run makes them."""
    G.gmg_timing_enable(ctx, True, as_launched=True)
    fn()
    out = {}
    for (kind, _, _), (n, _) in G.gmg_timing_table(ctx).items():
        out[kind] = out.get(kind, 0) + n
    G.gmg_timing_enable(ctx, False)
    return out


@pytest.mark.parametrize("prec", [0, 1])
def test_timing_as_launched(prec):
    import paper_1402_3545_amd as G
    w = W.SMALL
    ctx, _, _ = problem(w.nx, w.ny, w.nz, nlevels=w.nlevels, kv=w.kv, seed=w.seed,
                        kh_model=w.kh_model, prec_precond=prec)
    dt = torch.float64 if prec == 0 else torch.float32
    n = w.nx * w.ny * w.nz
    fd, u0 = (ctx.to_device(W.uniform_pm1(41, s, n), dtype=dt) for s in (1, 2))

    def cycle():
        ud = u0.clone()
        G.gmg_vcycle(ctx, fd, ud)
        outs.append(ctx.from_device(ud))

    outs = []
    cycle()
    kinds = _launched(G, ctx, cycle)
    down = ctx.nlevels - 1
    # the first smoothing step, the way down and up, the coarsest level's second step
    assert kinds == {"smooth": 2, "restrict_solve": down, "prolong_smooth": down}
    assert (outs[0] == outs[1]).all()
    # each fused kind by itself
    for kind in ("restrict_solve", "prolong_smooth"):
        G.gmg_timing_filter(ctx, [kind])
        G.gmg_timing_enable(ctx, True)
        cycle()
        table = G.gmg_timing_table(ctx)
        G.gmg_timing_enable(ctx, False)
        assert {(k[0], v[0]) for k, v in table.items()} == {(kind, 1)}
    G.gmg_timing_filter(ctx, None)
    with pytest.raises(G.GmgError):
        G.gmg_set_launch(ctx, "restrict_solve", 0, prec, 4, 0)


# entries on the coarse levels, and the kinds a V-cycle must then launch there
# (fused: without one of them)
ENTRIES = [({"line_solve": (1, 0), "smooth": (1, 0)},
            {"residual_restrict", "line_solve", "prolongate", "smooth"}),
           ({"line_solve": (1, 0)}, {"residual_restrict", "line_solve", "prolong_smooth"}),
           ({"smooth": (1, 0)}, {"restrict_solve", "prolongate", "smooth"}),
           ({"residual_restrict": (8, 0), "prolongate": (4, 2)},
            {"residual_restrict", "line_solve", "prolongate", "smooth"}),
           ({"residual_restrict": (4, 0), "prolongate": (4, 0), "line_solve": (4, 1),
             "smooth": (2, 4)}, {"restrict_solve", "prolong_smooth"})]


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("grid", [(64, 64, 64, 4), (40, 24, 37, 3), (96, 72, 128, 4)])
@pytest.mark.parametrize("entries,kinds", ENTRIES)
def test_cycle_runs_the_set_shapes(entries, kinds, grid, prec):
    """The kernels that the launch shapes ask for run whether they are timed or
    not; with cyclic reduction among them the cycle matches the oracle's like
    any other shape (the bars of the folded prolongation's tests), with the
    others it is bitwise that without entries."""
    import paper_1402_3545_amd as G
    nx, ny, nz, L = grid
    ctx, orc, _ = problem(nx, ny, nz, nlevels=L, seed=87, prec_precond=prec)
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    f, u = W.uniform_pm1(87, 1, n), W.uniform_pm1(87, 2, n)
    if prec == 1:
        f, u = (a.astype(np.float32).astype(np.float64) for a in (f, u))
    fd, u0 = ctx.to_device(f, dtype=dt), ctx.to_device(u, dtype=dt)

    def cycle():
        ud = u0.clone()
        G.gmg_vcycle(ctx, fd, ud)
        outs.append(ctx.from_device(ud))

    outs = []
    cycle()
    for kind, (rows, group) in entries.items():
        for lvl in range(L):
            # (the restriction is timed and shaped under the finer level; the
            # finest level's line kernels keep their defaults)
            if lvl > 0 or kind == "residual_restrict":
                G.gmg_set_launch(ctx, kind, lvl, prec, rows, group)
    cycle()
    # (the finest level's first step, the coarsest level's second one)
    got = set(_launched(G, ctx, cycle)) - {"smooth", "prolong_smooth"}
    assert got == kinds - {"smooth", "prolong_smooth"}
    G.gmg_timing_enable(ctx, True)
    cycle()
    G.gmg_timing_enable(ctx, False)
    assert all(np.array_equal(o, outs[1]) for o in outs[2:])
    if all(rows != 1 for rows, _ in entries.values()):
        assert np.array_equal(outs[0], outs[1])
    else:
        assert not np.array_equal(outs[0], outs[1])
    ref = orc.vcycle(f, u)
    assert max_rel(outs[1], ref, np.abs(ref).max()) < (1e-11 if prec == 0 else 1e-4)


def test_smoother_shape_above_the_block_forms():
    """Without an entry of the fold the FP64 post-smoother of a larger level
    takes the prolongation along; with one of the smoother it runs in that
    shape (bitwise the same cycle)."""
    import paper_1402_3545_amd as G
    nx, ny, nz = 192, 180, 20
    ctx, _, _ = problem(nx, ny, nz, nlevels=2, seed=88)
    n = nx * ny * nz
    fd, u0 = (ctx.to_device(W.uniform_pm1(88, s, n)) for s in (1, 2))
    outs, kinds = [], []

    def cycle():
        ud = u0.clone()
        G.gmg_vcycle(ctx, fd, ud)
        outs.append(ctx.from_device(ud))

    for shape in (None, (4, 0), (2, 4)):
        if shape:
            G.gmg_set_launch(ctx, "smooth", 0, G.GMG_F64, *shape)
        kinds.append(_launched(G, ctx, cycle))
    assert kinds[0].get("prolong_smooth") == 1 and "prolongate" not in kinds[0]
    for k in kinds[1:]:
        assert k.get("prolongate") == 1 and "prolong_smooth" not in k
    assert all(np.array_equal(o, outs[0]) for o in outs)


@pytest.mark.parametrize("prec", [0, 1])
def test_autotuner_on_small_levels(prec):
    """Levels of few columns have one kernel for every form but cyclic
    reduction, timed once: the table holds (4, 0) or (1, 0) for their line
    kernels and (4, 0) or (2, 0) for the fold, and the restriction is set
    apart from the line solve only by a shape that a kernel of its own has."""
    import paper_1402_3545_amd as G
    nx, ny, nz, L = 96, 64, 64, 4
    ctx, orc, _ = problem(nx, ny, nz, nlevels=L, seed=89, prec_precond=prec)
    G.gmg_autotune(ctx, reps=2)
    for lvl in range(L):
        assert G.gmg_get_launch(ctx, "line_solve", lvl, prec) in ((4, 0), (1, 0))
        assert G.gmg_get_launch(ctx, "smooth", lvl, prec) in ((4, 0), (1, 0))
        assert G.gmg_get_launch(ctx, "prolong_smooth", lvl, prec) in ((4, 0), (2, 0))
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    f, u = (W.uniform_pm1(89, s, n).astype(np.float32).astype(np.float64) for s in (1, 2))
    fd, ud = ctx.to_device(f, dtype=dt), ctx.to_device(u, dtype=dt)
    G.gmg_timing_enable(ctx, True, as_launched=True)
    G.gmg_vcycle(ctx, fd, ud)
    table = G.gmg_timing_table(ctx)
    G.gmg_timing_enable(ctx, False)
    for lvl in range(L - 1):
        apart = (G.gmg_get_launch(ctx, "residual_restrict", lvl, prec) != (4, 0) or
                 G.gmg_get_launch(ctx, "line_solve", lvl + 1, prec) == (1, 0))
        p = "f64" if prec == 0 else "f32"
        assert (("residual_restrict", lvl, p) in table) == apart
        assert (("restrict_solve", lvl, p) in table) != apart
    ref = orc.vcycle(f, u)
    assert max_rel(ctx.from_device(ud), ref, np.abs(ref).max()) < (1e-11 if prec == 0 else 1e-4)


@pytest.mark.parametrize("prec", [0, 1])
def test_launch_table_round_trip(prec):
    """A saved table gives the context it is applied to the kernels of the one
    it was read from, entries that nobody set included; clearing an entry
    brings the default back."""
    import paper_1402_3545_amd as G
    nx, ny, nz, L = 192, 180, 40, 2

    def context():
        return problem(nx, ny, nz, nlevels=L, seed=90, prec_precond=prec)[0]

    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz

    def launched(ctx):
        fd, ud = (ctx.to_device(W.uniform_pm1(90, s, n), dtype=dt) for s in (1, 2))
        return _launched(G, ctx, lambda: G.gmg_vcycle(ctx, fd, ud))

    a, b = context(), context()
    plain = launched(a)
    assert plain.get("prolong_smooth") == 1 and plain.get("restrict_solve") == 1
    assert G.launch_table(a) == {}
    G.apply_launch_table(b, G.launch_table(a))
    assert launched(b) == plain
    # (4, 0) is reported for an entry that nobody set, and is one when set
    assert G.gmg_get_launch(a, "smooth", 0, prec) == (4, 0)
    assert not G.gmg_launch_is_set(a, "smooth", 0, prec)
    G.gmg_set_launch(a, "smooth", 0, prec, 4, 0)
    G.gmg_set_launch(a, "line_solve", 1, prec, 1, 0)
    assert G.gmg_launch_is_set(a, "smooth", 0, prec)
    table = G.launch_table(a)
    assert table == {f"smooth/0/{prec}": [4, 0], f"line_solve/1/{prec}": [1, 0]}
    apart = launched(a)
    assert "prolong_smooth" not in apart and "restrict_solve" not in apart
    G.apply_launch_table(b, table)
    assert launched(b) == apart
    for c in (a, b):
        G.gmg_clear_launch(c, "smooth", 0, prec)
        G.gmg_clear_launch(c, "line_solve", 1, prec)
        assert G.launch_table(c) == {} and launched(c) == plain
    with pytest.raises(G.GmgError):
        G.gmg_clear_launch(a, "smooth", L, prec)
    with pytest.raises(G.GmgError):
        G.gmg_launch_is_set(a, 99, 0, prec)


@pytest.mark.parametrize("grid,prec,folded", [
    # FP64, ragged last tile: apart with more than 96 layers, up to 28672 columns
    ((136, 128, 128), 0, False), ((136, 128, 97), 0, False), ((136, 128, 96), 0, True),
    ((168, 168, 128), 0, False), ((176, 176, 128), 0, True), ((160, 128, 128), 0, True),
    # FP32 above 64 layers: apart up to 32768 columns
    ((136, 128, 128), 1, False), ((192, 172, 65), 1, True), ((136, 128, 64), 1, True)])
def test_where_the_fold_is_the_default(grid, prec, folded):
    """One kernel or two on the finest level without launch shapes: bitwise the
    cycle with the fold switched on and off."""
    import paper_1402_3545_amd as G
    nx, ny, nz = grid
    ctx, _, _ = problem(nx, ny, nz, nlevels=2, seed=92, prec_precond=prec)
    dt = torch.float64 if prec == 0 else torch.float32
    n = nx * ny * nz
    fd, u0 = (ctx.to_device(W.uniform_pm1(92, s, n), dtype=dt) for s in (1, 2))
    outs = []

    def cycle():
        ud = u0.clone()
        G.gmg_vcycle(ctx, fd, ud)
        outs.append(ctx.from_device(ud))

    kinds = _launched(G, ctx, cycle)
    assert ("prolong_smooth" in kinds) == folded and ("prolongate" in kinds) != folded
    for rows in (2, 4):
        G.gmg_set_launch(ctx, "prolong_smooth", 0, prec, rows, 0)
        cycle()
    assert all(np.array_equal(o, outs[0]) for o in outs[1:])
