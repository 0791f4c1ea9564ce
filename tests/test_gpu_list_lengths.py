"""Neighbour lists of every length: the kernels that know K = 4 and 8 when they are compiled and
the ones that take a run-time K (their wavefronts of several points stage the lists in LDS)
against the oracle, with dropped entries in the middle of a list and points that do not fill a
wavefront."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes
from tests.gpu_util import TOL, dev, gpu_plan, gpu_points, parity_err

pytestmark = pytest.mark.gpu


def lists(sc, n, k):
    """n x k lists as a caller may hand them over: repeated probes, entries out of range."""
    from paper_2510_07729_amd import sop
    g = np.random.default_rng(17 * n + k)
    idx = g.integers(0, sc.probe_pos.shape[0], (n, k)).astype(np.int32)
    idx[g.random((n, k)) < 0.2] = -1
    idx[g.random((n, k)) < 0.05] = 1 << 30
    w = (g.random((n, k)) / k).astype(np.float32)
    order = g.permutation(n).astype(np.int32)
    nb = sop.Neighbors(dev(order), dev(idx), dev(w))
    keep = idx < sc.probe_pos.shape[0]
    return nb, np.where(keep, idx, -1), w


@pytest.mark.parametrize("k", [1, 2, 3, 5, 7, 9, 12, 15, 16])
@pytest.mark.parametrize("n,S", [(1, 5), (67, 33), (201, 16)])
@pytest.mark.parametrize("half", [False, True])
def test_list_lengths(k, n, S, half):
    import torch

    from paper_2510_07729_amd import sop
    sc = scenes.tiny_shade(n_points=n, n_dirs=S, k=k, seed=n + k)
    if half:
        sc.texels = sc.texels.astype(np.float16).astype(np.float32)
    plan, pts = gpu_plan(sc), gpu_points(sc)
    tex, env = dev(sc.texels), dev(sc.env)
    tex = tex.half() if half else tex
    nb, idx, w = lists(sc, n, k)
    for how in (dict(), dict(rotate_per_point=True), dict(cosine=True)):
        rgb = sop.sop_shade(plan, tex, env, pts, S, nb=nb, seed=5, **how)
        ref = oracle.shade(sc, idx, w, n_dirs=S, seed=5, per_point=bool(how.get("rotate_per_point")),
                           cosine=bool(how.get("cosine")))
        assert parity_err(rgb.cpu().numpy(), ref).max() <= TOL, how
    sky = scenes.octahedral_sky(np.random.default_rng(1), 16)
    rgb, irr = sop.sop_shade(plan, tex, sop.OctEnv(dev(sky)), pts, S, nb=nb, seed=3,
                             env_sampling=True, irradiance=True)
    ref = oracle.shade_envis(sc, idx, w, n_dirs=S, seed=3, irradiance=True, env=sky)
    assert parity_err(rgb.cpu().numpy(), ref[0]).max() <= TOL
    assert parity_err(irr.cpu().numpy(), ref[1]).max() <= TOL
    ws = sop.workspace(plan._lib.sop_shadow_workspace_size(plan.handle, n, k, S, 16, 1), "cuda")
    for sampler in (0, 1):
        ref = oracle.shadow_ratio(sc.normal, sc.texels, idx, w, sky, S, seed=3,
                                  sampler=sampler)["ratio"]
        for room in (None, ws):                  # from occlusion maps, and from the maps
            out = sop.sop_shadow_ratio(plan, tex, dev(sky), pts, S, nb=nb, seed=3,
                                       sampler=sampler, ws=room)
            assert parity_err(out.cpu().numpy(), ref).max() <= TOL, (sampler, room is None)
