"""The sky estimates at the sizes where their lane layout changes (one, four or 16 points per
wavefront): sampled points against the oracle, and the same points in a call small enough
for another layout."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes
from tests.gpu_util import TOL, dev, gpu_plan, gpu_points, parity_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,S", [(1, 1), (5, 33), (61, 32), (59_999, 40), (60_001, 40),
                                 (1003, 16), (131_100, 2), (131_100, 34)])
@pytest.mark.parametrize("sampler", [0, 2])
def test_shadow_ratio(n, S, sampler):
    from paper_2510_07729_amd import sop
    sc = scenes.shadow_scene(n_points=n, n_probes=64, res=8, env_res=16, n_dirs=S, k=4)
    plan = gpu_plan(sc)
    z = dev(np.zeros(1, np.float32))
    pts = sop.Points(dev(sc.pos), dev(sc.normal), z, z, z)
    out = sop.sop_shadow_ratio(plan, dev(sc.texels), dev(sc.env), pts, S, k=4, seed=3,
                               sampler=sampler).cpu().numpy()
    rows = np.random.default_rng(n).choice(n, min(n, 500), replace=False)
    idx, w = oracle.knn(sc.probe_pos, sc.bounds_lo, sc.bounds_hi, sc.pos[rows], sc.normal[rows],
                        4)
    # without room for the occlusion maps the call reads the texels themselves
    ws = sop.workspace(plan._lib.sop_shadow_workspace_size(plan.handle, n, 4, S, 16, 0), "cuda")
    plain = sop.sop_shadow_ratio(plan, dev(sc.texels), dev(sc.env), pts, S, k=4, seed=3,
                                 sampler=sampler, ws=ws).cpu().numpy()
    half = [sop.sop_shadow_ratio(plan, dev(sc.texels).half(), dev(sc.env), pts, S, k=4, seed=3,
                                 sampler=sampler, ws=w).cpu().numpy() for w in (None, ws)]
    # sums of S terms of one sign in another order, and their quotient
    for a, b in ((out, plain), half):
        assert np.all(np.abs(a - b) <= 2.0 ** -22 * (S + 8) * np.abs(b))
    ref = oracle.shadow_ratio(sc.normal[rows], sc.texels, idx, w, sc.env, S, seed=3,
                              sampler=sampler, ids=rows)["ratio"]
    assert parity_err(out[rows], ref).max() <= TOL


@pytest.mark.parametrize("n,S", [(1, 1), (67, 33), (131_071, 16), (131_073, 16), (1003, 32)])
def test_relighting(n, S):
    import torch

    from paper_2510_07729_amd import sop
    sc = scenes.tiny_shade(n_points=n, res=8, n_dirs=S)
    sky = sop.OctEnv(dev(scenes.octahedral_sky(np.random.default_rng(1), 16)))
    plan, tex, pts = gpu_plan(sc), dev(sc.texels), gpu_points(sc)
    run = lambda p: sop.sop_shade(plan, tex, sky, p, S, k=4, seed=3, env_sampling="exact")
    rgb = run(pts)
    m = min(n, 2000)                            # the same points, keyed by the same indices
    part = run(sop.Points(*(x[:m].contiguous() for x in (pts.pos, pts.normal, pts.albedo,
                                                         pts.rough, pts.metal)),
                          view=pts.view[:m].contiguous()))
    # the draws are the same; only the order of the sums differs: S terms, all positive
    assert torch.all((rgb[:m] - part).abs() <= 2.0 ** -23 * (S + 8) * part.abs())
