"""bf16 attention of plans that keep every pair: their own kernel against the fp64 oracle and against the
windowed kernels (which a plan with a fixed patches_per_wave keeps).  Units of 32 rows and chunks of 64
keys at their edges, tiles across several scales, both workgroup sizes, every way to say "dense"."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu

# scales, query scales, B, H: one row more than a patch; units of 31, 32, 33 rows' worth; chunks of 63 to 65
# keys; sides out of order; tiles across scales; a generation step; 34 heads of 3000 rows take eight waves
CASES = [((1, 4), None, 2, 3), ((4, 4, 1), None, 2, 3), ((1, 2, 5), (1, 3), 2, 1), ((8,), None, 2, 2),
         ((1, 8), None, 2, 1), ((3, 7, 2, 6), None, 2, 3), ((1, 2, 3, 4, 5, 6), None, 2, 5),
         ((1, 2, 3, 4, 6, 9, 13), (5, 7), 2, 3), ((5, 12), (1, 2), 2, 1), ((11, 16), None, 4, 1),
         ((2, 10, 30, 44), None, 2, 17)]


def _close(a, b, ulps=3):
    """bf16 results of the same sums in another order, probabilities rounded to bf16 in between: the
    relative 2-norm stays below one bf16 rounding (2^-9) each and that of the probabilities."""
    a, b = a.float(), b.float()
    return float((a - b).norm()) <= ulps * 2.0 ** -9 * float(b.norm())


@pytest.mark.parametrize("scales,q_scales,B,H", CASES)
@pytest.mark.parametrize("scale", [1.0, 6.0])          # 6: peaked rows, the reference moves between blocks
def test_dense_kernel(scales, q_scales, B, H, scale):
    import paper_2411_17178_amd as lv
    q, k, v = workloads.make_qkv(scales, B, H, 64, "bf16", 7, 1.0, q_scales)
    q = (q.float() * scale).to(torch.bfloat16)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    plan = lv.litevar_mask_build(scales, -1, None, 0, q_scales)
    windowed = lv.litevar_mask_build(scales, -1, None, 0, q_scales, waves_per_group=(16, 0, 0, -1, 2))
    print(f"  dense: scales={scales} q_scales={q_scales} B={B} H={H} rows={plan.q_len}", flush=True)
    share = torch.tensor([[(h + s) % 2 for s in range(len(scales))] for h in range(H)], dtype=torch.uint8).cuda()
    got = lv.litevar_windowed_attn_fwd(plan, qd, kd, vd, 0.125)
    want = lv.litevar_windowed_attn_fwd(windowed, qd, kd, vd, 0.125)
    got_s = lv.litevar_windowed_attn_fwd(plan, qd, kd, vd, 0.125, cfg_share=share)
    want_s = lv.litevar_windowed_attn_fwd(windowed, qd, kd, vd, 0.125, cfg_share=share)
    torch.cuda.synchronize()
    assert _close(got, want) and _close(got_s, want_s)
    if plan.q_len <= 300:
        ref = oracle.attn(scales, oracle.expand_radii(scales, -1), *[workloads.to_oracle_array(t) for t in (q, k, v)],
                          0.125, 0, q_scales)
        assert np.abs(got.float().cpu().numpy() - ref).max() <= 2e-2      # the bf16 path's tolerance


def test_dense_by_other_means_and_layouts():
    """Sink scales over everything, windows that cover every part, bands as wide as their parts, one table
    per head: the same pairs, the same kernel, the same bits; tensors laid out [B, L, H, 64]."""
    import paper_2411_17178_amd as lv
    scales, B, H = (1, 2, 3, 5, 7), 2, 3
    K = len(scales)
    q, k, v = (t.cuda() for t in workloads.make_qkv(scales, B, H, 64, "bf16", 8, 1.0, None))
    want = lv.litevar_windowed_attn_fwd(lv.litevar_mask_build(scales, -1), q, k, v, 0.125)
    plans = [lv.litevar_mask_build(scales, 0, None, K), lv.litevar_mask_build(scales, 7),
             lv.litevar_mask_build(scales, 100, mask_mode=1),
             lv.litevar_mask_build(scales, 0, [[[7 + h] * K for _ in range(K)] for h in range(H)])]
    for plan in plans:
        assert torch.equal(lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125), want)
    by_token = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in (q, k, v)]
    assert torch.equal(lv.litevar_windowed_attn_fwd(plans[1], *by_token, 0.125), want)


def test_dense_rows_of_later_scales_do_not_reach_earlier_queries():
    import paper_2411_17178_amd as lv
    scales = (1, 2, 3, 5, 6)
    q, k, v = (t.cuda() for t in workloads.make_qkv(scales, 2, 2, 64, "bf16", 9, 1.0, None))
    plan = lv.litevar_mask_build(scales, -1)
    want = lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125)
    k[:, :, 39:], v[:, :, 39:] = float("nan"), float("nan")               # the last scale's rows
    got = lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125)
    assert torch.equal(got[:, :, :39], want[:, :, :39])


def test_dense_unusable_plan_leaves_the_output_alone():
    import paper_2411_17178_amd as lv
    scales = (1, 2, 3, 5)
    q, k, v = (t.cuda() for t in workloads.make_qkv(scales, 1, 2, 64, "bf16", 9, 1.0, None))
    n = lv.litevar_mask_plan_bytes(scales, -1)
    blob = torch.empty(n, dtype=torch.uint8, device="cuda")
    plan = lv.litevar_mask_build(scales, -1, blob=blob)
    blob.zero_()
    out = torch.full_like(q, 3.0)
    lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125, out=out)
    assert bool((out == 3.0).all())
