"""The sky estimates at both sides of every line of their rule for points per wavefront (32 draws;
65,536 points relit; 60,000 and, from the occlusion maps, 131,072 points with the ratio), with 7
and 8 draws (lists ordered by probe from 8 on) and lists of 4, 6 and 8 entries: points sampled
from the whole call, the last wavefront's among them, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes
from tests.gpu_util import TOL, dev, gpu_plan, gpu_points, parity_err

pytestmark = pytest.mark.gpu


def sample(n):
    rows = np.random.default_rng(n).choice(n, min(n, 400), replace=False)
    rows[:17] = np.arange(n - 17, n)
    return np.unique(rows)


@pytest.mark.parametrize("n,S,k", [(19, 7, 8), (1003, 32, 6), (1003, 33, 6), (65_535, 8, 8),
                                   (65_536, 8, 8), (65_536, 7, 4), (65_539, 32, 6),
                                   (65_539, 33, 4), (131_073, 16, 4)])
@pytest.mark.parametrize("exact", [False, True])
def test_relighting(n, S, k, exact):
    from paper_2510_07729_amd import sop
    sc = scenes.tiny_shade(n_points=n, res=8, n_dirs=S, k=k)
    sky = scenes.octahedral_sky(np.random.default_rng(1), 16)
    rgb, irr = sop.sop_shade(gpu_plan(sc), dev(sc.texels), sop.OctEnv(dev(sky)), gpu_points(sc), S,
                             k=k, seed=3, env_sampling="exact" if exact else True,
                             irradiance=True)
    rows = sample(n)
    idx, w = oracle.knn(sc.probe_pos, sc.bounds_lo, sc.bounds_hi, sc.pos[rows], sc.normal[rows], k)
    for key in ("pos", "normal", "view", "albedo", "rough", "metal"):
        setattr(sc, key, getattr(sc, key)[rows].copy())
    ref = oracle.shade_envis(sc, idx, w, n_dirs=S, seed=3, ids=rows, irradiance=True, env=sky,
                             exact=exact)
    assert parity_err(rgb.cpu().numpy()[rows], ref[0]).max() <= TOL
    assert parity_err(irr.cpu().numpy()[rows], ref[1]).max() <= TOL


@pytest.mark.parametrize("n,S,k", [(19, 7, 8), (1003, 32, 6), (59_999, 33, 8), (60_000, 33, 8),
                                   (60_003, 40, 6), (131_071, 8, 8), (131_072, 8, 8),
                                   (131_075, 33, 6), (131_072, 7, 4)])
@pytest.mark.parametrize("sampler", [0, 1])
def test_shadow_ratio(n, S, k, sampler):
    from paper_2510_07729_amd import sop
    sc = scenes.shadow_scene(n_points=n, n_probes=64, res=8, env_res=16, n_dirs=S, k=k)
    plan = gpu_plan(sc)
    z = dev(np.zeros(1, np.float32))
    pts = sop.Points(dev(sc.pos), dev(sc.normal), z, z, z)
    rows = sample(n)
    idx, w = oracle.knn(sc.probe_pos, sc.bounds_lo, sc.bounds_hi, sc.pos[rows], sc.normal[rows], k)
    ref = oracle.shadow_ratio(sc.normal[rows], sc.texels, idx, w, sc.env, S, seed=3,
                              sampler=sampler, ids=rows)["ratio"]
    ws = sop.workspace(plan._lib.sop_shadow_workspace_size(plan.handle, n, k, S, 16, 0), "cuda")
    for room in (None, ws):                      # from occlusion maps, and from the maps
        out = sop.sop_shadow_ratio(plan, dev(sc.texels), dev(sc.env), pts, S, k=k, seed=3,
                                   sampler=sampler, ws=room).cpu().numpy()
        assert parity_err(out[rows], ref).max() <= TOL, room is None
