"""The training kernel's 16-point tiles: batches below, at and just above one, two and more tiles,
with points that have no target mass, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2510_07729_amd import scenes
from tests.gpu_util import dev, gpu_points, log
from tests.test_gpu_proposal import OFF, batch, gpu_mlp, sop

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 15, 16, 17, 31, 33, 100])
def test_train_tiles_match_oracle(B):
    """Both sides round the same operands to bfloat16; an operand whose FP32 and FP64 values round
    to neighbouring numbers is off by 2^-8, so a group of gradients, every entry of which is a sum
    of products of two such operands, stays within 2^-7 in the L2 norm even if each of them were;
    bounded by 2^-6. The loss has no such operand past the logits."""
    log(f"training kernel: batch {B}")
    import torch
    sc, T = batch(B, seed=B)
    T[::7] = 0.0                                  # no mass: the uniform target
    params = scenes.mlp_init(seed=B)
    params[OFF["b1"]] = 0.05
    params[OFF["b2"]] = 0.05
    mlp = gpu_mlp(params, sc)
    grad = torch.full((params.size,), float("nan"), dtype=torch.float32, device="cuda")
    loss = sop().sop_proposal_train_step(mlp, gpu_points(sc), dev(T), grad=grad)
    g = grad.cpu().numpy().astype(np.float64)
    lo, go = oracle.mlp_loss_grad(params.astype(np.float64), sc.pos, sc.normal, sc.view, sc.rough,
                                  sc.bounds_lo, sc.bounds_hi, T, emulate_bf16=True)
    assert abs(float(loss.item()) - lo) <= 1e-4 * abs(lo)
    for name, sl in OFF.items():
        l2 = np.linalg.norm(g[sl] - go[sl]) / np.linalg.norm(go[sl])
        log(f"grad {name}: relative L2 {l2:.3e}")
        assert l2 <= 2.0 ** -6, name
