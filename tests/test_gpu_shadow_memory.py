"""Device memory of the shadow ratio: room for the maps' occlusion channel is asked for only by
calls that copy it out, and a call that does not get it still gives the same result."""
import gc

import numpy as np
import pytest

from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


def scene(P, R, n):
    import torch

    from paper_2510_07729_amd import sop
    g = torch.Generator(device="cuda")
    g.manual_seed(P + n)
    unit = lambda m: torch.nn.functional.normalize(
        torch.randn(m, 3, device="cuda", generator=g), dim=1)
    plan = sop.Plan(unit(P), np.full(3, -1.05, np.float32), np.full(3, 1.05, np.float32))
    tex = torch.rand(P, R, R, 4, device="cuda", generator=g)
    z = torch.zeros(1, device="cuda")
    x = unit(n)
    pts = sop.Points(x, x.clone(), z, z, z)
    return plan, tex, torch.rand(16, 16, 3, device="cuda", generator=g), pts


def test_no_room_for_small_calls():
    import torch

    from paper_2510_07729_amd import sop
    plan, tex, sky, pts = scene(2048, 64, 100)       # maps of 134 MB, their occlusion 36 MB
    run = lambda: sop.sop_shadow_ratio(plan, tex, sky, pts, 16, k=4)
    run()
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    run()
    assert torch.cuda.max_memory_allocated() - before < 4 << 20


def test_call_near_the_memory_limit():
    import torch

    from paper_2510_07729_amd import sop
    n, S, k = 300_000, 64, 4
    gc.collect()
    torch.cuda.empty_cache()                         # no free stretch of an earlier test
    plan, tex, sky, pts = scene(4096, 64, n)         # occlusion 71 MB, samples 1.08 times that
    need = plan._lib.sop_shadow_workspace_size(plan.handle, n, k, S, 16, 0)
    ref = sop.sop_shadow_ratio(plan, tex, sky, pts, S, k=k, ws=sop.workspace(need, "cuda"))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.mem_get_info()[1]
    room = torch.cuda.memory_reserved() + need + (44 << 20)   # the call's own needs, no more
    torch.cuda.set_per_process_memory_fraction(room / total)
    try:
        out = sop.sop_shadow_ratio(plan, tex, sky, pts, S, k=k)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(out, ref)


def test_more_occlusion_values_than_a_launch_has_threads():
    """65,536 half-precision maps of 256 x 256: 4.36e9 values, the last ones beyond 2^32; and
    as many samples, so that they are copied out."""
    import torch

    from paper_2510_07729_amd import sop
    gc.collect()
    torch.cuda.empty_cache()
    P, R, n, S = 65_536, 256, 1_100_000, 4096
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs 64 GiB of device memory")
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    unit = lambda m: torch.nn.functional.normalize(
        torch.randn(m, 3, device="cuda", generator=g), dim=1)
    plan = sop.Plan(unit(P), np.full(3, -1.05, np.float32), np.full(3, 1.05, np.float32))
    tex = torch.empty(P, R, R, 4, device="cuda", dtype=torch.float16)
    one = torch.rand(1024, R, R, 4, device="cuda", generator=g).half()
    for p in range(0, P, 1024):                      # every block of probes another occlusion
        tex[p:p + 1024] = one.roll(p // 1024, dims=1)
    z = torch.zeros(1, device="cuda")
    x = unit(n)
    pts = sop.Points(x, x.clone(), z, z, z)
    sky = torch.rand(16, 16, 3, device="cuda", generator=g)
    need = plan._lib.sop_shadow_workspace_size(plan.handle, n, 1, S, 16, 0)
    out = sop.sop_shadow_ratio(plan, tex, sky, pts, S, k=1)
    ref = sop.sop_shadow_ratio(plan, tex, sky, pts, S, k=1, ws=sop.workspace(need, "cuda"))
    # sums of S terms of one sign, the occlusion's four terms in another order
    assert bool(torch.all((out - ref).abs() <= 2.0 ** -22 * (S + 8) * ref.abs()))
    assert float((out - ref).abs().max()) < 1e-4     # a missing part of the maps is off by ~1
    del tex, one
    torch.cuda.empty_cache()
