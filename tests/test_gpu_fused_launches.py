"""The V-cycle's fused launches (restriction with the coarse line solve,
prolongation with the post-smoother): what is timed is what runs."""

import pytest

import workloads as W
from tests.gpu_util import problem

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
