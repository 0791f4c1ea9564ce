"""The bake at every line of its rule for lanes per ray: scenes whose rays meet few, some and
many candidates, calls of as many rays as the most that take 8 or 4 lanes and one probe more.
Which lanes trace a ray decides nothing, so every call gives the same bytes as the largest."""
import numpy as np
import pytest

from paper_2510_07729_amd import scenes
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,size", [(50, 0.02), (1000, 0.03), (1000, 0.3)])
@pytest.mark.parametrize("update", [False, True])
def test_lines_give_the_same_bytes(count, size, update):
    import torch

    from paper_2510_07729_amd import sop
    g = np.random.default_rng(count)
    unit = lambda n: scenes.unit_vectors(g, n)
    quat = g.standard_normal((count, 4))
    quat /= np.linalg.norm(quat, axis=1, keepdims=True)
    arrays = [unit(count) * 0.5 * (0.3 + g.random((count, 1))),
              np.exp(0.5 * g.standard_normal((count, 3))) * size, quat,
              0.3 + 0.7 * g.random(count), g.random((count, 3))]
    args = [dev(a.astype(np.float32)) for a in arrays]
    plan = sop.BakePlan(*args)
    if update:                                  # the rule stays that of the plan's creation
        args[1] = 0.8 * args[1]                 # smaller, so that they stay inside its grid
        plan.update(*args)
        plan.check()
    pos = dev((unit(2049) * 0.9).astype(np.float32))
    tex, dep = sop.sop_bake(plan, pos, 16)
    assert bool(torch.isfinite(tex).all())
    for n in (1, 128, 129, 256, 257, 512, 513, 768, 769, 2048):
        t, d = sop.sop_bake(plan, pos[:n].contiguous(), 16)
        assert torch.equal(t, tex[:n]) and torch.equal(d, dep[:n]), n
