"""Reads and readbacks at the size where a kernel's stores to pinned memory give
way to a copy (32,768 bytes): host reads return what was written, and a batch whose states take the copy steps like its pads alone."""
import numpy as np
import pytest

from gpu_util import gpu_pad, tc
from workloads import scenes

pytestmark = pytest.mark.gpu
MM = 1e-3


def _pad(cells):
    pad = scenes.box_pad(18 * MM, 14 * MM, 4 * MM, *cells)
    top = pad.X[pad.X[:, 2] >= 4 * MM - 1e-12]
    xy = top[np.argmin(np.hypot(top[:, 0] - 9 * MM, top[:, 1] - 7 * MM)), :2]
    ind = scenes.place_indenter(pad, scenes.SPHERE, xy, 1e-4, sphere_radius=4 * MM).at_depth(0.06 * MM)
    return pad, ind


# positions of 8, 1,365 (32,760 bytes) and 1,368 (32,832 bytes) vertices
@pytest.mark.parametrize("cells", [(1, 1, 1), (12, 14, 6), (17, 18, 3)])
def test_host_reads_return_what_was_written(cells):
    pad, ind = _pad(cells)
    ctx = tc.Context(0)
    gp = gpu_pad(ctx, pad, "mixed")
    st = gp.step([ind])
    assert np.array_equal(gp.read("reaction")[0], np.array(st.reaction))
    rng = np.random.default_rng(3)
    for _ in range(3):
        x, v = pad.X + 1e-6 * rng.standard_normal(pad.X.shape), rng.standard_normal(pad.X.shape)
        gp.write("positions", x)
        gp.write("velocities", v)
        assert np.array_equal(gp.read("positions"), x) and np.array_equal(gp.read("velocities"), v)
    # of one byte to an element (by default the bottom is fixed) and of four
    assert np.array_equal(gp.read("fixed") != 0, pad.X[:, 2] < 1e-12)
    assert np.array_equal(gp.read("tets"), pad.tets)
    gp.close()
    ctx.close()


def test_reads_after_another_call_failed():
    """A read reports its own errors, not the one that an earlier call of the
    thread left behind."""
    pad, ind = _pad((4, 3, 2))
    ctx = tc.Context(0)
    gp = gpu_pad(ctx, pad, "mixed")
    assert ctx.lib.hipSetDevice(1 << 20) != 0
    assert np.array_equal(gp.read("positions"), pad.X)
    assert ctx.lib.hipGetLastError() != 0      # (and clears it)
    gp.close()
    ctx.close()


def test_states_beyond_the_limit_are_copied():
    """130 pads' states take more than 32,768 bytes, 2 pads' do not."""
    ctx = tc.Context(0)
    pad, ind = _pad((4, 3, 2))
    few = [gpu_pad(ctx, pad, "mixed") for _ in range(2)]
    many = [gpu_pad(ctx, pad, "mixed") for _ in range(130)]
    for pads in (few, many):
        for _ in range(2):
            tc.step_batch(ctx, pads, [[ind]] * len(pads))
    ref = few[0].read("positions")
    assert not np.array_equal(ref, pad.X)
    for p in (few[1], many[0], many[64], many[-1]):
        assert np.array_equal(p.read("positions"), ref)
    for p in few + many:
        p.close()
    ctx.close()


def test_many_reports():
    """A report is whole whenever its flag is seen: 400 readings of alternating
    contents that fill the report, and batches on two streams, each pass of
    hundreds of state readbacks, that leave the same bits."""
    ctx = tc.Context(0)
    pad, ind = _pad((12, 14, 6))
    gp = gpu_pad(ctx, pad, "mixed")
    rng = np.random.default_rng(5)
    xs = [pad.X + 1e-6 * rng.standard_normal(pad.X.shape) for _ in range(2)]
    for k in range(400):
        gp.write("positions", xs[k % 2])
        assert np.array_equal(gp.read("positions"), xs[k % 2]), k
    gp.close()
    ctx.set_streams(2)
    cells = [(4, 3, 2), (11, 7, 5), (13, 14, 4), (20, 16, 5)] * 4
    made = [_pad(c) for c in cells]
    pads = [gpu_pad(ctx, p, "mixed", newton_tol=1e-8) for p, _ in made]
    ref = None
    for k in range(15):
        for p in pads:
            p.reset()
        tc.step_batch(ctx, pads, [[i] for _, i in made])
        x = [p.read("positions") for p in pads]
        ref = ref or x
        assert all(np.array_equal(a, b) for a, b in zip(ref, x)), k
    for p in pads:
        p.close()
    ctx.close()
