"""fp32 attention reads kept pairs only: a row of V that is not finite reaches the queries that keep its
key and no other one, in the step's other queries as little as in its padding."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu


# the key: one that several patches keep in part (windows), the first of a step with padding (it fills it), one
# of a plan with a single step per patch
@pytest.mark.parametrize("scales,radius,key", [((1, 2, 3, 5, 8), 1, 45), ((1, 2, 3, 5, 8), 1, 70), ((2, 9), 0, 40), ((1, 2, 3), 0, 7),
                                               ((1, 2, 3, 4, 5, 6, 8, 10, 13, 16), 2, 300), ((3, 17), 2, 9)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_value_row_that_is_not_finite(scales, radius, key, value):
    import paper_2411_17178_amd as lv
    q, k, v = workloads.make_qkv(scales, 1, 3, 64, "f32", 13, 1.0, None)
    radii = oracle.expand_radii(scales, radius)
    ref = oracle.attn(scales, radii, *[workloads.to_oracle_array(t) for t in (q, k, v)], 0.125, 0)
    keeps = oracle.mask_dense(scales, radii, 0)[:, key].astype(bool)
    assert keeps.any() and not keeps.all()
    v[:, 1, key, 5::7] = value                               # head 1, some dimensions
    plan = lv.litevar_mask_build(scales, radius)
    got = lv.litevar_windowed_attn_fwd(plan, q.cuda(), k.cuda(), v.cuda(), 0.125).cpu().numpy()
    hit = np.zeros(got.shape, dtype=bool)
    hit[:, 1, keeps, 5::7] = True
    assert np.abs(got[~hit] - ref[~hit]).max() <= 1e-5       # the path's tolerance
    assert not np.isfinite(got[hit]).any()
