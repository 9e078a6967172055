"""Results that do not move from version to version: the first CG iterate and whole
steps of single pads against the bits recorded in golden/step_bits.json.

Every sum of the solver is a fixed tree.  Its order is part of a step's result:
near convergence the line search compares energies that differ by their
rounding, so another order of r.z, right to its last bit, changes how often
Newton iterates and the stresses of a step in double by 1e-9.  The records come
from a version whose diagonal assembly finished a group's rows one after another in
a single lane; a version that must change them says so and records anew."""
import hashlib
import json
import os

import numpy as np
import pytest

from gpu_util import gpu_pad, tc
from workloads import scenes

pytestmark = pytest.mark.gpu
MM = 1e-3
RECORD = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "step_bits.json")

# rows: 8, 80, 240, 1050 (past one block's CG), 2142 and 17,220 (270 partials)
CELLS = [(1, 1, 1), (4, 3, 3), (7, 5, 4), (13, 14, 4), (20, 16, 5), (40, 34, 11)]


def _pressed(cells, depth=0.06 * MM):
    pad = scenes.box_pad(18 * MM, 14 * MM, 4 * MM, *cells)
    top = pad.X[pad.X[:, 2] >= 4 * MM - 1e-12]
    xy = top[np.argmin(np.hypot(top[:, 0] - 9 * MM, top[:, 1] - 7 * MM)), :2]
    return pad, scenes.place_indenter(pad, scenes.SPHERE, xy, 1e-4, sphere_radius=4 * MM).at_depth(depth)


def _shaken(gp, pad, seed=7):
    """Every vertex off its rest position, so that no row's gradient is zero."""
    x = pad.X + 1e-6 * np.random.default_rng(seed).standard_normal(pad.X.shape)
    x[pad.X[:, 2] < 1e-12] = pad.X[pad.X[:, 2] < 1e-12]
    gp.write("positions", x)


def _digest(*arrays):
    h = hashlib.sha256()
    for a in arrays:
        h.update(np.ascontiguousarray(a).tobytes())
    return h.hexdigest()[:16]


def iterate_bits(cells, prec):
    """d after one CG iteration, alpha z, at six positions (half of the time two
    orders of r.z agree to the last bit), and after four; with the gradients."""
    pad, ind = _pressed(cells)
    ctx = tc.Context(0)
    out = []
    for seed, its in ((1, 1), (2, 1), (3, 1), (4, 1), (5, 1), (6, 1), (7, 4)):
        gp = gpu_pad(ctx, pad, prec, quasi_static=1, cg_rel_tol=1e-14, cg_forcing=0, max_cg=its)
        _shaken(gp, pad, seed)
        out += gp.newton_direction([ind])
        gp.close()
    ctx.close()
    return _digest(*out)


def episode_bits(cells, prec, warm):
    pad, _ = _pressed(cells)
    ctx = tc.Context(0)
    gp = gpu_pad(ctx, pad, prec, newton_tol=1e-9, cg_warm=warm)
    _shaken(gp, pad)
    for depth in (0.1, 0.2):
        gp.step([_pressed(cells, depth * MM)[1]])
    out = _digest(*[gp.read(f) for f in ("positions", "sigma", "traction", "pressure")])
    gp.close()
    ctx.close()
    return out


def launch_bits(shape):
    """Vertex-row and SpMV blocks of other sizes, each with its own order of sums."""
    pad, ind = _pressed((40, 34, 11))
    ctx = tc.Context(0)
    ctx.set_launch(cg_block=shape[0], spmv_block=shape[1])
    gp = gpu_pad(ctx, pad, "fp64", quasi_static=1, cg_rel_tol=1e-14, cg_forcing=0, max_cg=4)
    _shaken(gp, pad)
    out = _digest(*gp.newton_direction([ind]))
    gp.close()
    ctx.close()
    return out


SHAPES = [(64, 64), (128, 256), (512, 512), (1024, 128)]


def all_bits():
    out = {}
    for prec in ("fp64", "mixed"):
        for cells in CELLS:
            out[f"iterate {cells} {prec}"] = iterate_bits(cells, prec)
        for cells in CELLS[:5]:
            for warm in (0, 1):
                out[f"episode {cells} {prec} {warm}"] = episode_bits(cells, prec, warm)
    for shape in SHAPES:
        out[f"launch {shape}"] = launch_bits(shape)
    return out


def _recorded(key):
    with open(RECORD) as f:
        return json.load(f)[key]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("cells", CELLS)
def test_cg_iterates_keep_their_bits(cells, prec):
    assert iterate_bits(cells, prec) == _recorded(f"iterate {cells} {prec}")


@pytest.mark.parametrize("warm", [0, 1])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("cells", CELLS[:5])
def test_steps_keep_their_bits(cells, prec, warm):
    assert episode_bits(cells, prec, warm) == _recorded(f"episode {cells} {prec} {warm}")


@pytest.mark.parametrize("shape", SHAPES)
def test_other_launch_shapes_keep_their_bits(shape):
    assert launch_bits(shape) == _recorded(f"launch {shape}")
