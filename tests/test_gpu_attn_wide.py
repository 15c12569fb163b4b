"""The 16-patch kernel's wide patches (32 queries per wave): shapes that tile sides of every remainder, both mask
modes, the order in which boxes are dealt, the moving softmax reference and operands that are not finite, against the
fp64 oracle (tolerance 2e-2: P and O are rounded to bf16) and against the sixteen-wave form of the same mask."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu
WIDE, NARROW = (16, 0, 0, -1, 2), (16, 0, 0, -1, 1)


@pytest.fixture(scope="module")
def lv():
    import paper_2411_17178_amd as m
    m.load_library()
    return m


def _ref(scales, radii, q, k, v, n_sink=0, q_scales=None, band=False):
    return oracle.attn(scales, radii, *[workloads.to_oracle_array(t) for t in (q, k, v)], 0.125, n_sink, q_scales,
                       mode=int(band))


def _run(lv, plan, q, k, v):
    o = lv.litevar_windowed_attn_fwd(plan, q.cuda(), k.cuda(), v.cuda(), 0.125)
    torch.cuda.synchronize()
    lv.litevar_plan_check(plan)                  # (the device's step counts equal the host's)
    return o.float().cpu().numpy()


# sides 1..8: one group, shapes from 1 x 1 to 4 x 8; 9, 10, 11, 13: 3 x 9, 5 x 5, 4 x 6, 4 x 7; 17, 19: 5 x 6 in groups of
# 20 x 12; 21: 7 x 4; 33: three columns of groups; 70: boxes wider than a wave
SHAPES = [((1, 2, 3, 4, 5, 6, 7, 8), 1), ((9, 10, 11), 2), ((3, 13, 14), 0), ((2, 17), 3), ((5, 19, 21), 2), ((33, 7), 4),
          ((1, 3, 70), 40), ((12, 25), -1), ((4, 9, 16), [2, 0, 5])]


@pytest.mark.parametrize("band", [False, True])
@pytest.mark.parametrize("scales,rad", SHAPES)
def test_every_patch_shape(lv, scales, rad, band):
    per = rad if isinstance(rad, list) else None
    radii = per or [rad] * len(scales)
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 31)
    out = {}
    for form in (WIDE, NARROW):
        plan = lv.litevar_mask_build(scales, 0 if per else rad, per, 1, waves_per_group=form, mask_mode=int(band))
        out[form] = _run(lv, plan, q, k, v)
    ref = _ref(scales, radii, q, k, v, 1, None, band)
    assert np.abs(out[WIDE] - ref).max() <= 2e-2
    assert np.abs(out[WIDE] - out[NARROW]).max() <= 2e-2


@pytest.mark.parametrize("shift", [-90.0, 0.0, 300.0])
def test_reference_follows_the_scores(lv, shift):
    """All scores of a query moved by one amount (in units of the exponent): the result does not change, although sums
    start below 2^-10, at 2^-11, or leave 2^40 on the way.  The amount grows over the scales, so that it keeps moving.
    Bound: the score is a sum of products of about |shift|, so the softmax weights carry 2^-9 |shift| / 8 of K's
    rounding at most; K's component is a power of two here, exact in bf16, and the bound is the usual one."""
    scales = (1, 2, 3, 4, 6, 9, 13, 18)
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 32)
    q[..., 0] = 8.0
    off = np.concatenate([[0], np.cumsum([s * s for s in scales])])
    for j in range(len(scales)):                 # the same for all keys of a scale
        k[:, :, off[j]:off[j + 1], 0] = 2.0 ** round(np.log2(abs(shift) + 1e-9)) * np.sign(shift) * (j + 1) / 8 if shift else 0.0
    plan = lv.litevar_mask_build(scales, 2, None, 0, (6, 8), waves_per_group=WIDE)
    lo = int(off[6])
    qs = q[:, :, lo:].contiguous()
    got = _run(lv, plan, qs, k, v)
    assert np.abs(got - _ref(scales, [2] * 8, qs, k, v, 0, (6, 8))).max() <= 2e-2


def test_scores_all_far_below_zero(lv):
    """Every kept score of every query at about -110 in base 2: sums would be 2^-107 at a reference of zero."""
    scales = (3, 5, 20)
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 33)
    q[..., 0], k[..., 0] = 8.0, -76.0            # 8 * -76 / 8 * log2(e) = -110
    plan = lv.litevar_mask_build(scales, 3, waves_per_group=WIDE)
    assert np.abs(_run(lv, plan, q, k, v) - _ref(scales, [3] * 3, q, k, v)).max() <= 2e-2


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("where", ["k", "v"])
def test_a_value_that_is_not_finite_reaches_the_queries_that_keep_it_only(lv, where, bad):
    scales, radius = (2, 4, 16), 1
    q, k, v = workloads.make_qkv(scales, 1, 2, 64, "bf16", 34)
    ref = _ref(scales, [radius] * 3, q, k, v)
    tok = 4 + 16 + 5 * 16 + 5                    # row 5, column 5 of the last scale
    (k if where == "k" else v)[0, 0, tok] = bad
    plan = lv.litevar_mask_build(scales, radius, waves_per_group=WIDE)
    got = _run(lv, plan, q, k, v)
    keeps = oracle.mask_dense(scales, [radius] * 3, 0)[:, tok].astype(bool)
    assert keeps.sum() == 9
    assert np.abs(got[0, 1] - ref[0, 1]).max() <= 2e-2 and np.abs(got[0, 0][~keeps] - ref[0, 0][~keeps]).max() <= 2e-2
    assert not np.isfinite(got[0, 0][keeps]).any()
