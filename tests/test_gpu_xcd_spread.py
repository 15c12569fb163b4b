"""Few (batch, head) pairs are dealt to several XCDs each: a call on the first heads of a batch gives, bit for
bit, what a call on 32 heads (one XCD per pair) gives for them, for every kernel that takes a plan apart."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


# one item (group) and several; heads that divide 8, that do not, and more than 8
@pytest.mark.parametrize("dtype,waves", [("bf16", 4), ("bf16", 8), ("bf16", (16, 0, 0, -1, 1)), ("bf16", (16, 0, 0, -1, 2)),
                                         ("f32", 4)])
@pytest.mark.parametrize("scales", [(1, 3), (1, 2, 5, 9, 20)])
def test_few_pairs_equal_many(dtype, waves, scales):
    import paper_2411_17178_amd as lv
    q, k, v = (t.cuda() for t in workloads.make_qkv(scales, 1, 32, 64, dtype, 5, 1.0, None))
    plan = lv.litevar_mask_build(scales, 2, waves_per_group=waves)
    want = lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125)
    for H in (1, 2, 3, 4, 5, 7, 9, 12, 20):
        print(f"  {dtype} waves={waves} scales={scales} H={H}", flush=True)
        got = lv.litevar_windowed_attn_fwd(plan, *(t[:, :H].contiguous() for t in (q, k, v)), 0.125)
        assert torch.equal(got, want[:, :H])
