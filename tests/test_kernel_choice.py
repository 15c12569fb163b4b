"""A plan whose options name a tiling of the windowed kernels runs on them, also where it keeps every pair."""
import pytest
import torch

import workloads


def test_handle_says_that_a_tiling_was_asked_for():
    import paper_2411_17178_amd as lv
    lv.load_library()
    for waves, chosen in ((0, 0), ((0, 0, 0, -1, 0), 0), (4, 1), (16, 1), ((0, 32, 0, -1, 0), 1), ((4, 0, 2, -1, 0), 1)):
        assert lv.litevar_mask_plan_stats((1, 2, 5), -1, waves_per_group=waves).tiling_chosen == chosen


@pytest.mark.gpu
@pytest.mark.parametrize("waves", [4, 8, 16, (4, 64, 2, 1), (8, 64, 2, 1)])
def test_dense_plan_with_a_tiling_runs_the_windowed_kernel(waves):
    """bit for bit what the same plan gives with a spin limit of its own, which has always kept that kernel; another
    order of sums than the default plan's"""
    import paper_2411_17178_amd as lv
    scales = (5, 9, 13)
    q, k, v = (t.cuda() for t in workloads.make_qkv(scales, 2, 40, 64, "bf16", 3, 1.0, None))
    got = [lv.litevar_windowed_attn_fwd(lv.litevar_mask_build(scales, -1, **kw), q, k, v, 0.125)
           for kw in (dict(waves_per_group=waves), dict(waves_per_group=waves, spin_limit=(1 << 22) + 1), {})]
    assert torch.equal(got[0], got[1]) and not torch.equal(got[0], got[2])
