"""A plan whose 32-query patches would need more than 65 535 steps runs with sixteen waves: 289 queries that keep
601 x 601 keys of each of three scales of side 1024, against fp32 products over all keys with a mask (2e-2 of the
largest result: P and O are rounded to bf16)."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_a_plan_without_wide_patches_runs():
    import paper_2411_17178_amd as lv
    scales, radius, side = (1024, 1024, 1024, 17), 300, 17
    plan = lv.litevar_mask_build(scales, radius, None, 0, (3, 4), waves_per_group=16)
    assert plan.patches_per_wave == 1
    lv.litevar_plan_check(plan)
    g = torch.Generator(device="cuda").manual_seed(61)
    q, k, v = (torch.randn((1, 1, n, 64), generator=g, device="cuda").to(torch.bfloat16)
               for n in (side * side, plan.kv_len, plan.kv_len))
    o = lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125)
    lv.litevar_plan_check(plan)
    want = torch.zeros((side * side, 64), device="cuda")
    total = torch.zeros((side * side, 1), device="cuda")
    at = 0
    for s in scales:                             # (N(0, 1) operands: no maximum needed in fp32)
        c = (2 * torch.arange(side, device="cuda") + 1) * s // (2 * side)
        near = (torch.arange(s, device="cuda")[None] - c[:, None]).abs() <= radius
        kept = (near[:, None, :, None] & near[None, :, None, :]).reshape(side * side, s * s)
        p = (q[0, 0].float() @ k[0, 0, at:at + s * s].float().T * 0.125).exp_() * kept
        want += p @ v[0, 0, at:at + s * s].float()
        total += p.sum(-1, keepdim=True)
        at += s * s
    scale = (want / total).abs().max().item()
    assert ((o[0, 0].float() - want / total).abs().max() <= 2e-2 * scale).item()      # (the mean of a million values)
