"""Farthest point sampling in rounds of many picks: the oracle's picks exactly, where rounds are
cut short or run over: one and several workgroups, few and many published points per
wavefront, clouds of ties and duplicates, more picks than distinct points."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes

pytestmark = pytest.mark.gpu


def cloud(kind, M, g):
    if kind == "ties":                          # integer lattice: whole shells tie
        n = int(np.ceil(M ** (1 / 3)))
        x = np.stack(np.meshgrid(*[np.arange(n)] * 3, indexing="ij"), -1).reshape(-1, 3)[:M]
    elif kind == "few":                         # 50 distinct places
        x = g.uniform(-1, 1, (50, 3))[g.integers(0, 50, M)]
    elif kind == "line":                        # every far point in one wavefront's share
        x = np.zeros((M, 3))
        x[: min(64, M), 0] = np.arange(min(64, M)) + 1.0
    else:
        x = g.uniform(-1, 1, (M, 3))
    return x.astype(np.float32)


@pytest.mark.parametrize("kind,M,P,start", [
    ("random", 1, 1, 0), ("random", 64, 64, 3), ("random", 255, 200, 254),
    ("random", 2048, 2048, 0),                  # one workgroup, every point picked
    ("random", 2049, 1500, 1),                  # two
    ("random", 20_000, 3000, 7),                # ten, 8 published points per wavefront
    ("random", 32_768, 2500, 5), ("random", 32_769, 2500, 5),   # 16 and 17: 8 and 4
    ("random", 140_001, 1500, 9),               # 64 workgroups, 9 points per thread
    ("random", 524_288, 300, 11),               # the largest cloud held in registers
    ("ties", 27_000, 1200, 0), ("ties", 40_000, 700, 39_999),
    ("few", 5000, 200, 4), ("few", 1000, 1000, 4), ("line", 9000, 300, 100),
])
def test_rounds_exact(kind, M, P, start):
    import torch

    from paper_2510_07729_amd import sop
    g = np.random.default_rng(M + P)
    x = cloud(kind, M, g)
    n = scenes.unit_vectors(g, M).astype(np.float32)
    pos, chosen = sop.sop_place_probes(torch.from_numpy(x).cuda(), torch.from_numpy(n).cuda(), P,
                                       start, 0.02)
    ref = oracle.fps(x, P, start)
    assert np.array_equal(chosen.cpu().numpy(), ref)
    assert np.array_equal(pos.cpu().numpy(), oracle.place(x, n, ref, 0.02))
