"""Calls whose work exceeds what one launch may hold (fewer than 2^32 threads)."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


# dtype, waves per group, scales, query scales, batch: each needs 2^32 threads or a little more; the inputs
# are broadcast over the batch (stride 0)
@pytest.mark.parametrize("dtype,waves,scales,q_scales,batch", [
    ("f32", 0, (1, 1), None, 524289),                       # one step per patch: 8 patches x 64 threads
    ("f32", 0, (6, 1), (1, 2), 262145),                     # two steps: 4 patches x 256 threads
    ("bf16", 4, (1,), None, 838865), ("bf16", 8, (1,), None, 466040),   # one group of 320 or 576 threads
    ("bf16", (16, 0, 0, -1, 1), (1,), None, 262145), ("bf16", (16, 0, 0, -1, 2), (1,), None, 524289),
    ("bf16", 0, (1,) * 17, None, 174765)])                  # all pairs kept: 3 tiles x 512 threads
def test_attention_of_more_threads_than_one_launch_holds(dtype, waves, scales, q_scales, batch):
    import paper_2411_17178_amd as lv
    H = 16
    print(f"  {dtype} waves={waves} scales={scales} pairs={batch * H}", flush=True)
    plan = lv.litevar_mask_build(scales, -1, None, 0, q_scales, waves_per_group=waves)
    q, k, v = (t.cuda() for t in workloads.make_qkv(scales, 1, H, 64, dtype, 3, 1.0, q_scales))
    want = lv.litevar_windowed_attn_fwd(plan, q, k, v, 0.125)
    out = torch.full((batch, H, plan.q_len, 64), 9.0, dtype=q.dtype, device="cuda")
    lv.litevar_windowed_attn_fwd(plan, *(t.expand(batch, -1, -1, -1) for t in (q, k, v)), 0.125, out=out)
    assert bool(out.eq(want).all())


@pytest.mark.parametrize("band", [False, True])
def test_calibration_of_more_threads_than_one_launch_holds(band):
    """65 535 heads x 262 slots x 256 threads, a map of 138 GB: every head has the same (uniform) map."""
    import paper_2411_17178_amd as lv
    scales, H = (1, 1, 1, 12, 11, 12, 11, 13) + (1,) * 24, 65535
    L = sum(s * s for s in scales)
    if torch.cuda.mem_get_info()[0] < 240e9:
        pytest.skip("needs 240 GB of free GPU memory")
    calibrate = lv.litevar_window_calibrate_band if band else lv.litevar_window_calibrate
    want = calibrate(scales, torch.ones((1, 1, L, L), device="cuda"), 0.8)
    print(f"  band={band} heads={H} L={L}", flush=True)
    got = calibrate(scales, torch.ones((1, H, L, L), device="cuda"), 0.8)
    assert torch.equal(got, want.expand_as(got))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def test_quantiser_of_more_rows_than_one_launch_holds():
    """2^29 + 70 rows, eight threads each: rows at both ends and where a second launch begins."""
    import paper_2411_17178_amd as lv
    rows, n = 2 ** 29 + 70, 200
    if torch.cuda.mem_get_info()[0] < 190e9:
        pytest.skip("needs 190 GB of free GPU memory")
    x = torch.zeros((rows, 64), dtype=torch.bfloat16, device="cuda")
    some = [slice(0, n), slice(2 ** 28, 2 ** 28 + n), slice(2 ** 29 - 2 * n, 2 ** 29 - n), slice(rows - n, rows)]
    for i, at in enumerate(some):
        x[at] = torch.randn((n, 64), generator=torch.Generator(device="cuda").manual_seed(i), device="cuda")
    codes, sz = lv.litevar_qkv8_quantize(x)
    back = lv.litevar_qkv8_dequantize(codes, sz)
    for at in some:
        want = lv.litevar_qkv8_quantize(x[at].contiguous())
        assert torch.equal(codes[at], want[0]) and torch.equal(sz[at], want[1])
        assert torch.equal(back[at], lv.litevar_qkv8_dequantize(*want))
    torch.cuda.synchronize()
    del x, codes, sz, back
    torch.cuda.empty_cache()
