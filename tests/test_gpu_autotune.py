"""The autotuner on batches whose CG runs in one block for all of the pads, or
for those left when the larger ones have ended."""
import numpy as np
import pytest

from gpu_util import gpu_pad, tc
from test_gpu_bits import _pressed

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [[(4, 3, 2), (7, 5, 4)], [(4, 3, 2), (20, 16, 5), (7, 5, 4), (4, 3, 3)]])
def test_small_and_mixed_batches(cells):
    ctx = tc.Context(0)
    made = [_pressed(c) for c in cells]
    pads = [gpu_pad(ctx, p, "mixed", newton_tol=1e-6) for p, _ in made]
    inds = [[i] for _, i in made]
    chosen = ctx.autotune(pads, inds)
    assert chosen[0] in (128, 256, 512, 1024) and chosen[2] in (128, 256, 512, 1024)
    assert chosen[1] in (64, 128, 256) and chosen[3] in (8, 12, 16, 24)
    for p, (q, _) in zip(pads, made):
        assert np.array_equal(p.read("positions"), q.X)
    assert all(s.status == 0 for s in tc.step_batch(ctx, pads, inds))
    for p in pads:
        p.close()
    ctx.close()
