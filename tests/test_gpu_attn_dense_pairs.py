"""The dense kernel's edge shapes with as many (batch, head) pairs as its dispatch asks for: small launches
of plans that keep every pair stay with the windowed kernels, so the shapes of test_gpu_attn_dense.py
are repeated here behind the rule's line, and once on its either side."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from test_gpu_attn_dense import CASES, _close

pytestmark = pytest.mark.gpu


def _dense(plan, pairs):
    """The library's rule: over 16 rows, and more windowed workgroups x steps per patch than 512, or over three steps."""
    patches = plan.n_patches * plan.n_head_groups
    return plan.q_len > 16 and (plan.n_steps > 3 * patches or pairs * plan.n_groups * plan.n_steps > 512 * patches)


def _enough(plan):
    """Heads for which a batch of two goes to the dense kernel."""
    H = 1
    while not _dense(plan, 2 * H):
        H += 1
    return H


def _inputs(scales, H, seed, q_scales=None, B=2):
    """Three distinct heads per batch row, repeated."""
    q, k, v = workloads.make_qkv(scales, B, 3, 64, "bf16", seed, 1.0, q_scales)
    return [t.repeat(1, -(-H // 3), 1, 1)[:, :H].contiguous() for t in (q, k, v)]


@pytest.mark.parametrize("scales,q_scales", [c[:2] for c in CASES[:-1]] +
                         [((1,) * 32, None), ((2, 1, 1, 3) * 8, (3, 30)), ((32, 1) * 4, (1, 8))])   # many scales
def test_dense_shapes(scales, q_scales):
    import paper_2411_17178_amd as lv
    plan = lv.litevar_mask_build(scales, -1, None, 0, q_scales)
    windowed = lv.litevar_mask_build(scales, -1, None, 0, q_scales, waves_per_group=(16, 0, 0, -1, 2))
    if plan.q_len <= 16:
        pytest.skip("one patch of rows stays with the windowed kernels")
    most = _enough(plan)
    for H in {most, max(1, most - 1)}:                     # the dense kernel's first, the windowed kernels' last
        print(f"  scales={scales} q_scales={q_scales} H={H} dense={_dense(plan, 2 * H)}", flush=True)
        q, k, v = _inputs(scales, H, 7, q_scales)
        qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
        share = torch.tensor([[(h + s) % 2 for s in range(len(scales))] for h in range(H)], dtype=torch.uint8).cuda()
        for more in ({}, {"cfg_share": share}):
            got = lv.litevar_windowed_attn_fwd(plan, qd, kd, vd, 0.125, **more)
            assert _close(got, lv.litevar_windowed_attn_fwd(windowed, qd, kd, vd, 0.125, **more))
        got = lv.litevar_windowed_attn_fwd(plan, qd, kd, vd, 0.125)
        n = min(H, 3)
        ref = oracle.attn(scales, oracle.expand_radii(scales, -1),
                          *[workloads.to_oracle_array(t[:, :n].contiguous()) for t in (q, k, v)], 0.125, 0, q_scales)
        assert np.abs(got[:, :n].float().cpu().numpy() - ref).max() <= 2e-2      # the bf16 path's tolerance
        assert torch.equal(got[:, n:], got[:, :n].repeat(1, -(-H // n), 1, 1)[:, n:H])   # repeated heads


def test_dense_by_other_means_and_layouts():
    import paper_2411_17178_amd as lv
    scales = (1, 2, 3, 5, 7)
    K, H = len(scales), _enough(lv.litevar_mask_build(scales, -1))
    q, k, v = (t.cuda() for t in _inputs(scales, H, 8))
    want = lv.litevar_windowed_attn_fwd(lv.litevar_mask_build(scales, -1), q, k, v, 0.125)
    plans = [lv.litevar_mask_build(scales, 0, None, K), lv.litevar_mask_build(scales, 7),
             lv.litevar_mask_build(scales, 100, mask_mode=1),
             lv.litevar_mask_build(scales, 0, [[[7 + h % 4] * K for _ in range(K)] for h in range(H)])]
    for plan in plans:
        assert _dense(plan, 2 * H)
        assert torch.equal(lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125), want)
    by_token = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v)]
    assert torch.equal(lv.litevar_windowed_attn_fwd(plans[1], *by_token, 0.125), want)


def test_dense_later_scales_and_unusable_plans():
    import paper_2411_17178_amd as lv
    scales = (1, 2, 3, 5, 6)
    blob = torch.empty(lv.litevar_mask_plan_bytes(scales, -1), dtype=torch.uint8, device="cuda")
    plan = lv.litevar_mask_build(scales, -1, blob=blob)
    H = _enough(plan)
    q, k, v = (t.cuda() for t in _inputs(scales, H, 9))
    want = lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125)
    k[:, :, 39:], v[:, :, 39:] = float("nan"), float("nan")               # the last scale's rows
    assert torch.equal(lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125)[:, :, :39], want[:, :, :39])
    torch.cuda.synchronize()
    blob.zero_()
    out = torch.full_like(q, 3.0)
    lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125, out=out)
    assert bool((out == 3.0).all())


@pytest.mark.parametrize("side,H", [(12, 299), (12, 300), (16, 300), (17, 300)])   # 5, 8 and 10 units of a 1168-key call
def test_dense_one_pass_of_eight_waves(side, H):
    import paper_2411_17178_amd as lv
    scales = (32, side)
    plan = lv.litevar_mask_build(scales, -1, None, 0, (1, 2))
    q, k, v = _inputs(scales, H, 7, (1, 2), B=1)
    got = lv.litevar_windowed_attn_fwd(plan, q.cuda(), k.cuda(), v.cuda(), 0.125).float().cpu()
    ref = oracle.attn(scales, oracle.expand_radii(scales, -1), *[workloads.to_oracle_array(t[:, :3].contiguous()) for t in (q, k, v)],
                      0.125, 0, (1, 2))
    assert np.abs(got[:, :3].numpy() - ref).max() <= 2e-2
    assert torch.equal(got[:, 3:], got[:, :3].repeat(1, -(-H // 3), 1, 1)[:, 3:H])
