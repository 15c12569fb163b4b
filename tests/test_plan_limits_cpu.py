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
