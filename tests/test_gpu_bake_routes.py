"""The bake by how many rays a call has (8, 4 or 2 lanes trace one ray), and the registration of
flat and long Gaussians in grids of different cells: which lanes test a Gaussian and in which
cells it is registered never decides what a ray resolves, so the bytes are the same."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes
from tests.gpu_util import TOL, dev, log, parity_err, report

pytestmark = pytest.mark.gpu


def bake(gs, probes, res, **opts):
    from paper_2510_07729_amd import sop
    plan = sop.BakePlan(dev(gs.mean), dev(gs.scale), dev(gs.rotation), dev(gs.opacity),
                        dev(gs.color), **opts)
    plan.check()
    tex, dep = sop.sop_bake(plan, dev(probes), res)
    return tex.cpu().numpy(), dep.cpu().numpy()


@pytest.mark.parametrize("probes,res", [(512, 16), (513, 16), (2048, 16), (2049, 16), (900, 11),
                                        (4000, 9), (9000, 9)])
def test_bake_routes_give_the_same_bytes(probes, res):
    """Calls at both sides of the limits (131,072 and 524,288 rays, padded to whole 8x8 tiles),
    whole and ragged tiles; the first and last 40 probes are baked again in calls of their own,
    which the eight-lane kernel takes."""
    log(f"bake: {probes} probes of {res}x{res} texels against calls of 40")
    rng = np.random.default_rng(probes + res)
    gs = scenes.random_gaussians(rng, 300)
    pos = rng.uniform(-0.5, 0.5, (probes, 3)).astype(np.float32)
    tex, dep = bake(gs, pos, res)
    for part in (slice(0, 40), slice(probes - 40, probes)):
        t, d = bake(gs, pos[part], res)
        assert np.array_equal(t, tex[part]) and np.array_equal(d, dep[part])
    assert np.isfinite(tex).all() and np.isfinite(dep).all()


@pytest.mark.parametrize("ratio", [30.0, 1000.0])
def test_bake_registers_flat_and_long_gaussians(ratio):
    """Scales apart by `ratio` along one axis (flat) or two (long), boxes from a fraction of a
    cell to thousands of cells: grids of small, default and single cells give the same bytes,
    and the rays agree with the oracle, which knows no grid."""
    log(f"bake: scale ratio {ratio:g}, four grids")
    rng = np.random.default_rng(int(ratio))
    gs = scenes.random_gaussians(rng, 240, log_scale=(-2.2, 0.7))
    thin = rng.integers(0, 3, gs.count)
    gs.scale[np.arange(gs.count), thin] /= np.float32(ratio)
    long = rng.random(gs.count) < 0.5
    gs.scale[np.flatnonzero(long), (thin[long] + 1) % 3] /= np.float32(ratio)
    pos = rng.uniform(-0.6, 0.6, (6, 3)).astype(np.float32)
    t0, d0 = bake(gs, pos, 16)
    for cs in (0.05, 0.7, 1000.0):
        t, d = bake(gs, pos, 16, cell_scale=cs)
        assert np.array_equal(t, t0) and np.array_equal(d, d0), cs
    rp = np.repeat(np.arange(6), 256).astype(np.int32)
    rt = np.tile(np.arange(256), 6).astype(np.int32)
    ref, amb = oracle.bake_rays(gs, pos.astype(np.float64), 16, rp, rt)
    keep = ~amb
    log(f"{amb.sum()} of {len(amb)} rays ambiguous (excluded)")
    err = parity_err(t0.reshape(-1, 256, 4)[rp, rt][keep], ref[keep, :4])
    assert report("rgbo", err) <= TOL
