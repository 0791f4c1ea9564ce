"""Neighbour search on both sides of the line between its kernels (a wavefront per point up to
1536 points per cell of a grid's side, a lane per point above), which the sizes here are taken
from: clamped points, finite radii, points far from all probes, boxes that grow over an empty
grid. Exact against the oracle, and equal bit for bit to the same points in calls small enough
for the other kernel."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_knn import HI, LO, cloud

pytestmark = pytest.mark.gpu


def place(kind, n, g):
    if kind == "far":                          # one small patch beside the sphere
        return (np.float32(-0.9) + 0.02 * g.random((n, 3))).astype(np.float32)
    if kind == "volume":
        return (2.0 * g.random((n, 3)) - 1.0).astype(np.float32)
    return cloud(kind, n, g)


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("P,K,probes,points,radius", [
    (30, 8, "sphere", "corner", np.inf),        # boxes grow over the whole grid
    (64, 16, "far", "sphere", np.inf),          # steps of more than a cell, most cells empty
    (64, 3, "sphere", "outside", 0.9),          # clamped points beyond and within the radius
    (64, 4, "sphere", "corner", 0.05),          # nothing within the radius
    (300, 5, "outside", "sphere", 0.2),         # lists with gaps
    (1000, 8, "far", "sphere", 1.5),            # the radius ends the growth
    (4096, 8, "sphere", "outside", np.inf),
    (4096, 8, "volume", "volume", 0.1),
])
def test_both_routes(P, K, probes, points, radius, over):
    import torch

    from paper_2510_07729_amd import sop
    g = np.random.default_rng(P * 7 + K)
    pp = place(probes, P, g)
    dev = lambda a: torch.from_numpy(a).cuda()
    plan = sop.Plan(dev(pp), LO, HI)
    _, dims, _ = plan.info()
    line = 1536 * int(dims[0])                  # the largest call of a wavefront per point
    N = line + over
    x, nrm = place(points, N, g), cloud("sphere", N, g)
    zero = torch.zeros(1, device="cuda")
    knn = lambda a, b: sop.sop_knn(plan, sop.Points(dev(x[a:b]), dev(nrm[a:b]), zero, zero, zero),
                                   K, radius)
    nb = knn(0, N)
    idx, w = nb.idx.cpu().numpy(), nb.w.cpu().numpy()
    rows = g.choice(N, 2000, replace=False)
    ridx, rw = oracle.knn(pp, LO, HI, x[rows], nrm[rows], K, radius)
    assert np.array_equal(idx[rows], ridx)
    gap = np.sqrt(((pp[np.maximum(ridx, 0)] - x[rows][:, None].astype(np.float64)) ** 2).sum(-1))
    gap = np.where(ridx < 0, np.inf, gap).min(1, keepdims=True)
    tol = 2.0 ** -24 * (32 + 8 / np.maximum(gap, 1e-7))   # as in the other search tests
    assert np.all(np.abs(w[rows] - rw) <= tol)
    if over:
        step = line // 3 + 1                    # three calls below the line
        for a in range(0, N, step):
            part = knn(a, min(N, a + step))
            assert torch.equal(part.idx, nb.idx[a:a + step])
            assert torch.equal(part.w, nb.w[a:a + step])
