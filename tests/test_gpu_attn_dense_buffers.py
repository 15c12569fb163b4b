"""Dense kernel: one to five chunks of 64 keys, whole and ragged, through each number of waves and LDS buffers that its
rule picks, against the fp64 oracle (tolerance 2e-2), and scores that move the softmax reference."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu


def _check(scales, H, q_scales, tune=None):
    import paper_2411_17178_amd as lv
    q, k, v = workloads.make_qkv(scales, 1, 3, 64, "bf16", 41, 1.0, q_scales)
    if tune:
        tune(q, k)
    ref = oracle.attn(scales, [-1] * len(scales), *[workloads.to_oracle_array(t) for t in (q, k, v)], 0.125, 0, q_scales)
    many = [t.repeat(1, -(-H // 3), 1, 1)[:, :H].contiguous().cuda() for t in (q, k, v)]
    plan = lv.litevar_mask_build(scales, -1, None, 0, q_scales)
    o = lv.litevar_windowed_attn_fwd(plan, *many, 0.125)
    torch.cuda.synchronize()
    o = o.float().cpu().numpy()
    assert np.abs(o[0, :3] - ref[0]).max() <= 2e-2
    for i in range(3):                           # the same head gives the same bits, wherever it ran
        assert (o[0, i::3] == o[0, i]).all()


# rows of the last scale; keys 50, 64, 113, 128, 130, 192, 196, 281, 337
SIZES = [(5, 5), (1, 3, 7, 2), (8, 7), (8, 8), (9, 7), (8, 8, 8), (14,), (16, 5), (16, 9)]


@pytest.mark.parametrize("H", [60, 1100])        # up to and beyond 512 workgroups of four waves
@pytest.mark.parametrize("scales", SIZES)
def test_chunks(scales, H):
    _check(scales, H, (len(scales) - 1, len(scales)))


@pytest.mark.parametrize("scales,H", [((13,), 200), ((16, 13), 130), ((24, 16), 420), ((5, 12), 384), ((5, 12), 385)])
def test_waves(scales, H):
    _check(scales, H, (len(scales) - 1, len(scales)))


@pytest.mark.parametrize("shift", [-76.0, 32.0, 256.0])
def test_reference_follows_the_scores(shift):
    """One amount on all scores of a scale (exact in bf16), growing over the scales: the first block lies far below zero, or sums pass 2^40."""
    scales = (6, 7, 9, 11)

    def tune(q, k):
        q[..., 0] = 8.0
        at = 0
        for j, s in enumerate(scales):
            k[:, :, at:at + s * s, 0] = shift * (j + 1) if shift > 0 else shift
            at += s * s
    _check(scales, 60, None, tune)
