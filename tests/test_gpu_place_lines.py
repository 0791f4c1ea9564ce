"""Farthest point sampling at both sides of the lines of its launch: 1024 points per workgroup,
8 published points per wavefront up to 16 workgroups and 4 above, and from 64 workgroups on 8,
16 and 32 points per thread. The oracle's picks exactly."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [256, 257, 512, 513, 1024, 1025, 16_384, 16_385, 65_536, 65_537,
                               131_072, 131_073, 262_144, 262_145])
def test_lines_exact(M):
    import torch

    from paper_2510_07729_amd import sop
    g = np.random.default_rng(M)
    x = g.uniform(-1, 1, (M, 3)).astype(np.float32)
    x[M // 2:] = x[: M - M // 2]                # pairs of equal points
    n = scenes.unit_vectors(g, M).astype(np.float32)
    P, start = min(M, 400), M // 3
    pos, chosen = sop.sop_place_probes(torch.from_numpy(x).cuda(), torch.from_numpy(n).cuda(), P,
                                       start, 0.02)
    ref = oracle.fps(x, P, start)
    assert np.array_equal(chosen.cpu().numpy(), ref)
    assert np.array_equal(pos.cpu().numpy(), oracle.place(x, n, ref, 0.02))
