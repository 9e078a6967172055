"""Which CG path ran, by the kernels' launch counts, and how many iterations
each is said to have done, at the limits of the one-block path and where it
takes over a solve that launched iterations began."""
import numpy as np
import pytest

from gpu_util import gpu_pad, tc
from test_gpu_bits import _pressed
from workloads import meshes, scenes

pytestmark = pytest.mark.gpu
MM = 1e-3


def _launches(ctx):
    t = ctx.timing()
    return {k: t[k][1] if k in t else 0 for k in ("cg_small", "cg_spmv", "cg_update")}


# rows: 8, 640 and 648 (the limit in float64), 1024 and 1050 (in mixed precision)
@pytest.mark.parametrize("prec,cells,small", [
    ("fp64", (1, 1, 1), True), ("fp64", (9, 7, 7), True), ("fp64", (8, 8, 7), False),
    ("mixed", (8, 8, 7), True), ("mixed", (15, 7, 7), True), ("mixed", (13, 14, 4), False)])
def test_path_by_rows(prec, cells, small):
    pad, ind = _pressed(cells)
    ctx = tc.Context(0)
    ctx.set_timing(1)
    gp = gpu_pad(ctx, pad, prec)
    gp.step([ind])
    n = _launches(ctx)
    gp.close()
    ctx.close()
    assert (n["cg_small"] > 0) == small and (n["cg_spmv"] > 0) == (not small) == (n["cg_update"] > 0), n


@pytest.mark.parametrize("why", ["wide rows", "other blocks"])
def test_launched_for_other_reasons(why):
    ctx = tc.Context(0)
    if why == "wide rows":
        X, T = meshes.fan_prisms(24, 6 * MM, 3 * MM, 2)
        pad = scenes.Pad("fan", X, T, scenes.Material(), (12 * MM, 12 * MM, 3 * MM))
        ind = scenes.place_indenter(pad, scenes.SPHERE, (0.0, 0.0), 1e-4, sphere_radius=4 * MM).at_depth(0.06 * MM)
    else:
        pad, ind = _pressed((4, 3, 2))
        ctx.set_launch(spmv_block=128)
    ctx.set_timing(1)
    gp = gpu_pad(ctx, pad, "mixed")
    gp.step([ind])
    n = _launches(ctx)
    gp.close()
    ctx.close()
    assert n["cg_small"] == 0 and n["cg_spmv"] > 0 and n["cg_update"] > 0, n


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("warm", [0, 1])
def test_one_block_takes_over_a_launched_solve(prec, warm):
    """A larger pad at rest ends its step while a small one is in its first
    solve: the launched iterations end there, one block goes on with it, with
    the bits of the pad alone, and the byte counts divide the iterations as
    they were run."""
    R = 8 if prec == "fp64" else 4
    small, ind = _pressed((7, 5, 4))
    large, _ = _pressed((20, 16, 5))
    kw = dict(cg_rel_tol=1e-12 if prec == "fp64" else 1e-6, cg_forcing=0, cg_warm=warm, newton_tol=1e-7)
    ctx = tc.Context(0)
    ctx.set_launch(cg_per_replay=2)
    alone = gpu_pad(ctx, small, prec, **kw)
    alone.step([ind])
    pads = [gpu_pad(ctx, small, prec, **kw), gpu_pad(ctx, large, prec, cg_rel_tol=0.5, cg_conv_tol=0.5)]
    ctx.set_timing(1)
    st = tc.step_batch(ctx, pads, [[ind], []])
    t = ctx.timing()
    ctx.set_timing(0)
    same = [np.array_equal(alone.read(f), pads[0].read(f)) for f in ("positions", "sigma")]

    def per_iteration(p):
        V = len(p.X)
        pairs = (p.tets[:, :, None].astype(np.int64) * V + p.tets[:, None, :]).ravel()
        nb = len(np.unique(pairs))      # blocks: vertices that share a tet
        return nb * (9 * R + 4) + 12 * R * V, V * (21 * R + 48)

    (bs, us), (bl, ul) = (per_iteration(p) for p in (small, large))
    launched = t["cg_spmv"][1]          # the small pad is in its first solve during each
    total = {k: t[k][1] * t[k][2] for k in ("cg_small", "cg_spmv", "cg_update")}
    for p in [alone] + pads:
        p.close()
    ctx.close()
    print("small", st[0], "large", st[1], "launched", launched, "small launches", t["cg_small"][1], flush=True)
    assert all(same)
    assert launched > 0 and t["cg_small"][1] > 0
    assert total["cg_small"] == pytest.approx((st[0].cg_iters - launched) * (bs + us), rel=1e-12)
    assert total["cg_spmv"] == pytest.approx(launched * bs + st[1].cg_iters * bl, rel=1e-12)
    assert total["cg_update"] == pytest.approx(launched * us + st[1].cg_iters * ul, rel=1e-12)
