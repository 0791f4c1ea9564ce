"""Rounding of the roughness gradient: no part of it is shared by all samples.

One probe per point with weight 1 and a constant map (occlusion 1), so that a point's gradient
is the material term of one sample times the looked-up radiance, which the albedo gradient has
as a factor too (metallic 1: spec (1 - x^5)): its rounding drops out of the difference of the
two relative errors. What is left are unbiased float32 roundings: over N = 200,000 points the
median has a standard error of 1.25 x 2e-7 / sqrt(N) = 6e-10. A constant or a scale that is
rounded by itself (a float 1/pi: 4e-8, a float 2 pi: 3e-8) shifts every point the same way."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes
from tests.gpu_util import dev, gpu_plan, gpu_points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("res", [8, 64])             # the batched and the general adjoint
def test_no_shared_rounding(res, deterministic):
    from paper_2510_07729_amd import sop
    n, S = 200_000, 1
    sc = scenes.tiny_shade(n_points=n, n_dirs=S, k=1, res=res, seed=9)
    sc.texels[:] = 1.0
    sc.env[:] = 0.0
    sc.metal[:] = 1.0
    idx, w = np.zeros((n, 1), np.int32), np.ones((n, 1), np.float32)
    nb = sop.Neighbors(dev(np.arange(n, dtype=np.int32)), dev(idx), dev(w))
    grad = np.ones((n, 3), np.float32)
    g = sop.sop_shade_backward(gpu_plan(sc), dev(sc.texels), dev(sc.env), gpu_points(sc),
                               dev(grad), S, nb=nb, seed=5, rotate_per_point=True,
                               deterministic=deterministic)
    ref = oracle.shade_backward(sc, idx, w.astype(np.float64), grad.astype(np.float64), seed=5,
                                per_point=True)
    rough = g["rough"].cpu().numpy() / ref["g_rough"] - 1.0
    albedo = (g["albedo"].cpu().numpy() / ref["g_albedo"] - 1.0)[:, 0]
    print(f"median {np.median(rough):.2e} and {np.median(albedo):.2e}, of the difference "
          f"{np.median(rough - albedo):.2e}", flush=True)
    assert abs(np.median(rough - albedo)) <= 4e-9
