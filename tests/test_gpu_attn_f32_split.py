"""fp32 attention: a patch's steps are dealt to four waves whose partial softmax results are merged
(fewer steps than waves, one each, remainders), against the fp64 oracle at the path's 1e-5."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu

# scales, radius, sink scales, query scales: 1 key; 1 step; 2, 3, 4, 5 steps and more per patch, with a
# short last step; patches cut by the grid's edge; a generation step
CASES = [((1,), 0, 0, None), ((2, 3), 0, 0, None), ((3, 5), -1, 0, None), ((1, 9), -1, 0, None),
         ((4, 11), -1, 1, (1, 2)), ((1, 2, 3, 4, 12), -1, 0, None), ((5, 7, 13), 2, 1, None),
         ((7, 11, 17), -1, 0, (2, 3)), ((2, 6, 9), 1, 0, (1, 2))]


@pytest.mark.parametrize("scales,radius,sink,q_scales", CASES)
@pytest.mark.parametrize("scale", [1.0, 6.0])          # 6: peaked rows, the reference moves between steps
def test_f32_steps_split_over_waves(scales, radius, sink, q_scales, scale):
    import paper_2411_17178_amd as lv
    q, k, v = workloads.make_qkv(scales, 2, 3, 64, "f32", 11, 1.0, q_scales)
    q = q * scale
    share = torch.tensor([[(h + s) % 2 for s in range(len(scales))] for h in range(3)], dtype=torch.uint8)
    plan = lv.litevar_mask_build(scales, radius, None, sink, q_scales)
    kd, vd = k.cuda(), v.cuda()
    if q_scales is not None:                               # cache rows behind the step's scales are never read
        end = plan.q_token_begin + plan.q_len
        kd[:, :, end:], vd[:, :, end:] = float("nan"), float("nan")
    radii = oracle.expand_radii(scales, radius)
    arrs = [workloads.to_oracle_array(t) for t in (q, k, v)]
    ref = oracle.attn(scales, radii, *arrs, 0.125, sink, q_scales)
    got = lv.litevar_windowed_attn_fwd(plan, q.cuda(), kd, vd, 0.125).cpu().numpy()
    assert np.abs(got - ref).max() <= 1e-5
    got = lv.litevar_windowed_attn_fwd(plan, q.cuda(), kd, vd, 0.125, cfg_share=share.cuda()).cpu().numpy()
    first, last = (0, len(scales)) if q_scales is None else q_scales
    row = 0
    for s in range(first, last):
        n = scales[s] ** 2
        for h in range(3):
            uncond = ref[0, h] if share[h, s] else ref[1, h]
            assert np.abs(got[0, h, row:row + n] - ref[0, h, row:row + n]).max() <= 1e-5
            assert np.abs(got[1, h, row:row + n] - uncond[row:row + n]).max() <= 1e-5
        row += n
