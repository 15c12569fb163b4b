"""Descriptors whose 32-query patches would need more than 65 535 steps, the limit of a patch: their boxes are larger than
those of the patches of 16.  Such plans are built without them, and the handle says so."""
import pytest

import paper_2411_17178_amd as lv

BIG = (1024, 1024, 1024)


@pytest.mark.parametrize("pw", [0, 1, 2])
@pytest.mark.parametrize("scales,radius", [(BIG + (17,), 300), (BIG + (17,), 320), (BIG + (32,), 360), ((512,) * 16 + (20,), 130)])
def test_plans_without_wide_patches(scales, radius, pw):
    K = len(scales)
    st = lv.litevar_mask_plan_stats(scales, radius, None, 0, (K - 1, K), waves_per_group=(16, 0, 0, -1, pw))
    assert st.patches_per_wave == 1 and st.waves_per_group == 16 and st.n_steps > 65535
    assert lv.litevar_mask_plan_bytes(scales, radius, None, 0, (K - 1, K), waves_per_group=(16, 0, 0, -1, pw)) == st.blob_bytes


@pytest.mark.parametrize("pw", [0, 1, 2])
def test_other_plans_say_what_was_asked(pw):
    for _ in range(2):                           # (the second from what the first one's sizing left)
        st = lv.litevar_mask_plan_stats((1, 4, 9, 24), 3, waves_per_group=(16, 0, 0, -1, pw))
        assert st.patches_per_wave == pw


def test_the_limit_itself_stays():
    with pytest.raises(lv.LitevarError):
        lv.litevar_mask_plan_stats(BIG + (16,), -1, None, 0, (3, 4), waves_per_group=16)


@pytest.mark.parametrize("scales,radius,q_scales,before", [
    ((1, 2, 3, 4, 5, 6, 8, 10, 13, 16), 3, (9, 10), 134400), ((1, 2, 3, 4, 6, 9, 13, 18, 24, 32), 4, None, 1427456),
    ((1, 2, 3, 4, 6, 9, 13, 18, 24, 32, 48, 64, 96, 128), 4, None, 37830144), ((1, 2, 3, 4, 6, 9, 13, 18, 24, 32), -1, None, 4721920)])
def test_size_of_plans_of_16_patches(scales, radius, q_scales, before):
    """before: the bytes of the same plan while its list was walked in steps of 16 queries alone.  A step of 32 takes 1024
    bytes instead of the 512 of each of its two, and serves up to 1.2 times the pairs: a tenth more in all."""
    plain = lv.litevar_mask_plan_stats(scales, radius, None, 0, q_scales, waves_per_group=(16, 0, 0, -1, 1))
    wide = lv.litevar_mask_plan_stats(scales, radius, None, 0, q_scales, waves_per_group=16)
    assert (wide.n_steps, wide.n_union_keys) == (plain.n_steps, plain.n_union_keys)
    assert plain.blob_bytes <= before and wide.blob_bytes <= 1.15 * before
