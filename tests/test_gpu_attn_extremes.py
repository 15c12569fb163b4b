"""Finite operands at the ends of their range through the 32-query kernel and the dense kernel, against the fp64
oracle.  Inputs are chosen so that scores are exact in fp32; outputs are compared relative to the largest value
(2e-2: P and O are rounded to bf16)."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu
WIDE = (16, 0, 0, -1, 2)


def _compare(scales, radii, q, k, v, sm_scale=0.125, q_scales=None, band=False, tol=2e-2, **build):
    import paper_2411_17178_amd as lv
    plan = lv.litevar_mask_build(scales, 0, radii, 0, q_scales, mask_mode=int(band), **build)
    o = lv.litevar_windowed_attn_fwd(plan, q.cuda(), k.cuda(), v.cuda(), sm_scale)
    torch.cuda.synchronize()
    lv.litevar_plan_check(plan)
    o = o.double().cpu().numpy()
    ref = oracle.attn(scales, radii, *[workloads.to_oracle_array(t) for t in (q, k, v)], float(np.float32(sm_scale)), 0, q_scales,
                      mode=int(band))
    assert np.isfinite(o).all()
    assert np.abs(o - ref).max() <= tol * max(1e-38, float(v.double().abs().max()))


@pytest.mark.parametrize("band", [False, True])
@pytest.mark.parametrize("case", ["product", "scale"])
def test_masked_pairs_stay_masked(case, band):
    """Raw products close to 2^128 with keys that few queries keep; a softmax scale of 9e-39."""
    scales, radii = (2, 5, 18), [2, 2, 2]
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 51)
    q[..., 0], k[..., 0] = 2.0 ** 61, 0.0
    if case == "product":
        for tok in (3, 17, 29 + 8 * 18 + 9, 29 + 200):
            k[:, :, tok, 0] = 1.9375 * 2.0 ** 66
    else:
        q[..., 0] = 0.0
    _compare(scales, radii, q, k, v, 0.125 if case == "product" else 9e-39, None, band, waves_per_group=WIDE)


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("form", ["dense", "wide", "band"])
def test_scores_beyond_the_reference(form, sign):
    """All of a query's scores equal and beyond 2^24 in base 2, where a reference in whole numbers, or rounded, is off
    by many powers of two: every head at a magnitude of its own, from 2^24 to 2^38; and a last scale that lies above or
    below the others by a part of it."""
    scales, H = (3, 6, 18), 36
    q, k, v = workloads.make_qkv(scales, 1, H, 64, "bf16", 54)
    q[..., 1:], k[..., 1:] = 0.0, 0.0
    for h in range(H):
        x = 2.0 ** (14 + h % 12) * (1 + h / 64)
        q[:, h, :, 0] = x
        k[:, h, :, 0] = sign * 2.0 ** 14
        if h >= 24:
            k[:, h, 9:45, 0] = sign * 2.0 ** 13
    build = {} if form == "dense" else {"waves_per_group": WIDE}
    _compare(scales, [-1 if form == "dense" else 3] * 3, q, k, v, band=form == "band", **build)


def _rising(scales, step):
    """K's component 0 grows by `step` from scale to scale (q's is 8, the softmax scale 1/8): scores rise by that much."""
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 52)
    q[..., 0] = 8.0
    at = 0
    for j, s in enumerate(scales):
        k[:, :, at:at + s * s, 0] = step * j
        at += s * s
    return q, k, v


@pytest.mark.parametrize("form", ["dense", "wide"])
def test_large_values_under_rising_scores(form):
    """Scores that rise by 24 (2^35 in the probabilities) over values of 2^105: sums of 2^35 would overflow in the products."""
    scales = (6, 7, 9, 11)
    q, k, v = _rising(scales, 8.0)
    v = (v.float().sign() * 2.0 ** 105 + 0.0).to(torch.bfloat16)
    _compare(scales, [-1 if form == "dense" else 3] * 4, q, k, v, **({"waves_per_group": WIDE} if form == "wide" else {}))


@pytest.mark.parametrize("level", [-26.0, -20.0, -10.0, -3.0])
@pytest.mark.parametrize("exponent", [-115, -122])
def test_small_values_under_low_scores(exponent, level):
    """Values of about 2^-115 under probabilities of 2^-37 would lose their bits in the products."""
    scales = (3, 5, 20)
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 53)
    q[..., 0], k[..., 0] = 8.0, level
    v = (v.float() * 2.0 ** exponent).to(torch.bfloat16)
    _compare(scales, [3] * 3, q, k, v, waves_per_group=WIDE)


@pytest.mark.parametrize("first,step", [(-44.0, 4.0), (-44.0, -4.0), (-100.0, 12.0)])
def test_low_scores_that_rise_or_fall(first, step):
    """Scores at -63 (-144) in base 2 from the first step on, higher or lower from scale to scale."""
    scales = (1, 2, 3, 4, 6, 9, 13, 18)
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 56)
    q[..., 0] = 8.0
    at = 0
    for j, s in enumerate(scales):
        k[:, :, at:at + s * s, 0] = first + step * j
        at += s * s
    _compare(scales, [2] * 8, q, k, v, waves_per_group=WIDE)


@pytest.mark.parametrize("band", [False, True])
@pytest.mark.parametrize("level", [-76.0, -28.0, 60.0])
def test_queries_that_keep_nothing_in_the_first_step(level, band):
    """The first key scale has the queries' own side: the queries of a patch's last rows keep none of the first step's 32 keys,
    while those of its first rows have their reference already."""
    scales = (20, 20)
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 57)
    q[..., 0], k[..., 0] = 8.0, level
    _compare(scales, [8, 8] if band else [1, 1], q[:, :, 400:].contiguous(), k, v, 0.125, (1, 2), band, waves_per_group=WIDE)
