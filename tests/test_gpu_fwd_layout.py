"""Shading forward at the sizes where its wavefronts are ragged: points that do not fill the
8 of a wavefront, directions that leave a pair of lanes half idle, lists with dropped
entries, per-point rotations. Oracle parity by the metric of the other shading tests."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes
from tests.gpu_util import TOL, gpu_plan, gpu_points, parity_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 7, 9, 33, 65])
@pytest.mark.parametrize("S,k,rotate,radius", [(1, 4, False, np.inf), (7, 8, True, np.inf),
                                               (9, 8, False, 0.3), (16, 3, True, 0.25),
                                               (37, 4, False, 0.2)])
def test_ragged_wavefronts(n, S, k, rotate, radius):
    import torch

    from paper_2510_07729_amd import sop
    sc = scenes.tiny_shade(n_points=n, n_dirs=S, k=k, seed=n + S)
    rgb, irr = sop.sop_shade(gpu_plan(sc), torch.from_numpy(sc.texels).cuda(),
                             torch.from_numpy(sc.env).cuda(), gpu_points(sc), S, k=k, seed=5,
                             radius=radius, rotate_per_point=rotate, irradiance=True)
    idx, w = oracle.knn(sc.probe_pos, sc.bounds_lo, sc.bounds_hi, sc.pos, sc.normal, k, radius)
    ref = oracle.shade(sc, idx, w, n_dirs=S, seed=5, per_point=rotate, irradiance=True)
    assert parity_err(rgb.cpu().numpy(), ref[0]).max() <= TOL
    assert parity_err(irr.cpu().numpy(), ref[1]).max() <= TOL
