"""The bounds-checking build on the dense kernel: nothing found and nothing changed on the library's own plans,
four and eight waves per workgroup; a handle that understates the cache by one token (the tensors hold it)
is reported."""
import pytest
import torch

import workloads
from test_gpu_debug_bounds import debug_lib, lv  # noqa: F401  (fixtures)

pytestmark = pytest.mark.gpu


# the second and fourth with eight waves; full sequences, generation steps, many scales
@pytest.mark.parametrize("scales,q_scales,H", [((1, 2, 5, 9, 12), None, 24), ((1, 2, 5, 9, 12), None, 200), ((1, 2, 3, 4, 5, 6, 8, 10, 13), (8, 9), 9),
                                               ((1, 2, 3, 4, 5, 6, 8, 10, 13, 16), (9, 10), 160), ((1, 3) * 16, (2, 31), 40)])
def test_checked_build_finds_nothing_on_dense_plans(lv, debug_lib, scales, q_scales, H):
    q, k, v = (t.cuda() for t in workloads.make_qkv(scales, 2, H, 64, "bf16", 5, 1.0, q_scales))
    share = workloads.make_cfg_share(H, len(scales), 9).cuda()
    plan = lv.litevar_mask_build(scales, -1, None, 0, q_scales)
    print(f"  checked build: scales={scales} q_scales={q_scales} H={H}", flush=True)
    want = lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125, cfg_share=share)
    with lv.use_library(debug_lib):
        got = lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125, cfg_share=share)
        torch.cuda.synchronize()
        lv.litevar_plan_check(plan)
    assert torch.equal(got, want)


@pytest.mark.parametrize("field,rows", [("kv_len", "k"), ("q_len", "q")])
def test_checked_build_reports_an_understated_length(lv, debug_lib, field, rows):
    scales, H = (1, 2, 5, 9), 60
    q, k, v = (t.cuda() for t in workloads.make_qkv(scales, 2, H, 64, "bf16", 5, 1.0, None))
    plan = lv.litevar_mask_build(scales, -1)
    out = torch.empty_like(q)
    setattr(plan.handle, field, getattr(plan.handle, field) - 1)
    if rows == "k":
        k, v = k[:, :, :-1], v[:, :, :-1]                 # views: the last row is still there
    else:
        q, out = q[:, :, :-1], out[:, :, :-1]
    with lv.use_library(debug_lib):
        lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125, out=out)
        torch.cuda.synchronize()
        with pytest.raises(lv.LitevarError, match="out of range"):
            lv.litevar_plan_check(plan)
