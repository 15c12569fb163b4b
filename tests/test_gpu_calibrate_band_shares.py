"""Band calibration of large scales, whose rows are dealt to 17 to 31 workgroups (remainders, the cap), against
sums by distance in numpy: the sums to 64-bit rounding, the radii exactly where the ratio is no tie."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scales,samples", [((33,), 2), ((40,), 1), ((1, 2, 3, 45), 3), ((64,), 1), ((1, 1, 1, 63), 5)])
def test_band_row_shares(scales, samples):
    import paper_2411_17178_amd as lv
    off = np.concatenate([[0], np.cumsum([s * s for s in scales])])
    L, r0 = int(off[-1]), 0.8
    p = torch.rand((samples, 1, L, L), generator=torch.Generator().manual_seed(3)) ** 3
    print(f"  scales={scales} samples={samples}", flush=True)
    rad, mass = lv.litevar_window_calibrate_band(scales, p.cuda(), r0, with_mass=True)
    total = p.double().sum(0).numpy()[0]
    for k in range(len(scales)):
        for first, last in [(0, min(2, k))] + [(j, j) for j in range(3, k + 1)]:
            block = total[off[k]:off[k + 1], off[first]:off[last + 1]]
            nk, n = block.shape
            dist = np.abs(np.arange(n)[None] - ((2 * np.arange(nk) + 1) * n // (2 * nk))[:, None])
            want = np.cumsum(np.bincount(dist.ravel(), weights=block.ravel(), minlength=n))
            got = mass[0, k, first, :n].cpu().numpy()
            assert np.abs(got - want).max() <= 1e-11 * want[-1]      # (2^24 terms of one sign at most, 2^-53 each, pairwise or in runs)
            ratio = want / want[-1]
            assert np.abs(ratio - r0).min() > 1e-9
            assert int(rad[0, k, first]) == int(np.argmax(ratio >= r0))
