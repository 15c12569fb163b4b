"""Threshold 1 of both calibrations at the edges of the prefix sums' runs of sixteen: the radius is the last distance
that holds any mass, exactly, because distances without mass add nothing to a sum."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _centre_distance(n_q, n_k):
    return np.abs(np.arange(n_k)[None] - ((2 * np.arange(n_q) + 1) * n_k // (2 * n_q))[:, None])


@pytest.mark.parametrize("side,last", [(4, 7), (4, 8), (5, 12), (16, 15), (16, 16), (16, 127), (17, 143), (64, 2047)])
def test_band_threshold_one(side, last):
    import paper_2411_17178_amd as lv
    n = side * side
    p = torch.rand((2, 1, n, n), generator=torch.Generator().manual_seed(side)) + 0.5
    p *= torch.from_numpy(_centre_distance(n, n) <= last)
    print(f"  side={side} last={last}", flush=True)
    rad, mass = lv.litevar_window_calibrate_band((side,), p.cuda(), 1.0, with_mass=True)
    assert int(rad[0, 0, 0]) == last
    m = mass[0, 0, 0].cpu().numpy()
    assert (np.diff(m) >= 0).all() and (m[last:] == m[-1]).all()
    assert abs(m[-1] / float(p.double().sum()) - 1) <= 1e-11       # (2^25 terms of one sign at most, 2^-53 each, in runs)


@pytest.mark.parametrize("side,last", [(15, 6), (16, 0), (17, 8), (33, 15), (33, 16), (64, 31)])
def test_window_threshold_one(side, last):
    import paper_2411_17178_amd as lv
    d = _centre_distance(side, side)
    keep = np.maximum(d[:, None, :, None], d[None, :, None, :]).reshape(side * side, side * side) <= last
    p = (torch.rand((1, 1) + keep.shape, generator=torch.Generator().manual_seed(side)) + 0.5) * torch.from_numpy(keep)
    print(f"  side={side} last={last}", flush=True)
    rad, mass = lv.litevar_window_calibrate((side,), p.cuda(), 1.0, with_mass=True)
    assert int(rad[0, 0, 0]) == last
    m = mass[0, 0, 0, :side].cpu().numpy()
    assert (np.diff(m) >= 0).all() and (m[last:] == m[-1]).all()
    assert abs(m[-1] / float(p.double().sum()) - 1) <= 1e-11
