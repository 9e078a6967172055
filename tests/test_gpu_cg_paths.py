"""The CG's paths on the GPU: pads whose whole solve runs in one block (up to
1024 rows in mixed precision, 640 in float64, rows of at most 16 blocks) and
pads whose iterations are launched, at the edges of the row steps, of the
limits and of the partial sums, against the oracle's exact Newton direction
and against each other."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla

from gpu_util import gpu_pad, log, oracle_pad, tc
from oracle import stepper
from workloads import meshes, scenes

pytestmark = pytest.mark.gpu
MM = 1e-3


def _pressed(cells):
    """A pad of nx x ny x nz cells under a sphere, a state near contact."""
    pad = scenes.box_pad(18 * MM, 14 * MM, 4 * MM, *cells)
    top = pad.X[:, 2] >= 4 * MM - 1e-12
    xy = pad.X[top][np.argmin(np.hypot(pad.X[top, 0] - 9 * MM, pad.X[top, 1] - 7 * MM)), :2]
    ind = scenes.place_indenter(pad, scenes.SPHERE, xy, 1e-4, sphere_radius=4 * MM).at_depth(0.06 * MM)
    return pad, ind


def _exact(pad, ind, prm):
    op = oracle_pad(pad)
    g = stepper.gradient(op, op.x, op.x, [ind], prm).ravel()
    H = stepper.hessian(op, op.x, [ind], prm)
    free = op.free.ravel()
    p = np.zeros(g.size)
    p[free] = spla.spsolve(H[free][:, free].tocsc(), -g[free])
    return p.reshape(-1, 3)


# rows: 8 (one cell), 60 and 80 around one row step of 64, 576 and 640 at nine
# and ten steps, 648 and 660 past the float64 limit, 1001 and 1050 around the
# mixed one
@pytest.mark.parametrize("cells", [(1, 1, 1), (4, 3, 2), (4, 3, 3), (11, 7, 5), (9, 7, 7), (8, 8, 7), (10, 9, 5),
                                   (12, 10, 6), (13, 14, 4)])
@pytest.mark.parametrize("prec,rel,tol", [("fp64", 1e-12, 1e-7), ("mixed", 1e-6, 2e-3)])
def test_direction_matches_oracle_at_the_edges(cells, prec, rel, tol):
    pad, ind = _pressed(cells)
    prm = stepper.StepParams(newton_tol=1e-10, quasi_static=True)
    ref = _exact(pad, ind, prm)
    ctx = tc.Context(0)
    gp = gpu_pad(ctx, pad, prec, quasi_static=1, cg_rel_tol=rel, cg_forcing=0)
    d, _ = gp.newton_direction([ind])
    err = np.abs(d - ref).max() / np.abs(ref).max()
    log(f"{cells} V {pad.X.shape[0]} {prec}: direction err {err:.2e}")
    ctx.close()
    assert err < tol


def test_wide_rows_are_launched():
    """A small pad whose rows exceed 16 blocks (an axis vertex of a disc of 24
    sectors) takes the launched iterations."""
    X, T = meshes.fan_prisms(24, 6 * MM, 3 * MM, 2)
    pad = scenes.Pad("fan", X, T, scenes.Material(), (12 * MM, 12 * MM, 3 * MM))
    ind = scenes.place_indenter(pad, scenes.SPHERE, (0.0, 0.0), 1e-4, sphere_radius=4 * MM).at_depth(0.06 * MM)
    prm = stepper.StepParams(newton_tol=1e-10, quasi_static=True)
    ref = _exact(pad, ind, prm)
    ctx = tc.Context(0)
    gp = gpu_pad(ctx, pad, "fp64", quasi_static=1, cg_rel_tol=1e-12, cg_forcing=0)
    assert gp.info["ell_width"] > 16 and gp.info["n_verts"] <= 640
    d, _ = gp.newton_direction([ind])
    ctx.close()
    assert np.abs(d - ref).max() / np.abs(ref).max() < 1e-7


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("warm", [0, 1])
def test_small_pads_in_a_mixed_batch_keep_their_bits(prec, warm):
    """Beside a larger pad the small ones' iterations are launched; alone each
    runs its solve in one block.  Same rows, sums and order: same bits."""
    ctx = tc.Context(0)
    out = {}
    for key in ("alone", "batch"):
        pads, inds = [], []
        for cells in ((4, 3, 2), (11, 7, 5), (9, 7, 7), (20, 16, 5)):
            pad, ind = _pressed(cells)
            pads.append(gpu_pad(ctx, pad, prec, cg_warm=warm))
            inds.append(ind)
        for _ in range(2):
            if key == "alone":
                for p, i in zip(pads, inds):
                    p.step([i])
            else:
                tc.step_batch(ctx, pads, [[i] for i in inds])
        out[key] = [(p.read("positions"), p.read("sigma")) for p in pads]
        for p in pads:
            p.close()
    ctx.close()
    for a, b in zip(out["alone"], out["batch"]):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("sectors", [40, 300])
def test_long_runs_of_edge_records(sectors):
    """The axis edges of a fan are shared by every sector's tets: runs of
    records below and beyond the 127 that a wave holds at a time in float64."""
    X, T = meshes.fan_prisms(sectors, 6 * MM, 3 * MM, 2)
    pad = scenes.Pad("fan", X, T, scenes.Material(), (12 * MM, 12 * MM, 3 * MM))
    ind = scenes.place_indenter(pad, scenes.SPHERE, (0.0, 0.0), 1e-4, sphere_radius=4 * MM).at_depth(0.06 * MM)
    ref = _exact(pad, ind, stepper.StepParams(newton_tol=1e-10, quasi_static=True))
    ctx = tc.Context(0)
    gp = gpu_pad(ctx, pad, "fp64", quasi_static=1, cg_rel_tol=1e-12, cg_forcing=0)
    d, _ = gp.newton_direction([ind])
    ctx.close()
    assert np.abs(d - ref).max() / np.abs(ref).max() < 1e-7


def test_partial_sums_shared_over_the_block():
    """More than 512 partials of a dot product are summed by the whole block:
    on 17k rows, products of 64-thread blocks leave 1,077 partials, those of
    256-thread blocks 270; a vector kernel of 256 threads takes the 1,077 in one
    round of loads, one of 64 in three.  All solve to 1e-10; the directions
    differ by what the solver leaves, far below 1e-6."""
    pad, ind = _pressed((40, 34, 11))
    d = []
    for cg_block, spmv_block in ((256, 256), (256, 64), (64, 64)):
        ctx = tc.Context(0)
        ctx.set_launch(cg_block=cg_block, spmv_block=spmv_block)
        gp = gpu_pad(ctx, pad, "fp64", quasi_static=1, cg_rel_tol=1e-10, cg_forcing=0)
        d.append(gp.newton_direction([ind])[0])
        ctx.close()
    for other in d[1:]:
        assert np.abs(d[0] - other).max() < 1e-6 * np.abs(d[0]).max()
