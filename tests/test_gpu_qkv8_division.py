"""The quantiser's quotients come from a reciprocal per row and two corrections; the codes are those of the
IEEE division the oracle makes, bit for bit: ties and their neighbours at many scales, and the rows whose
scale is too small or too large for the short form."""
import numpy as np
import pytest
import torch

import oracle
import workloads

pytestmark = pytest.mark.gpu


def _rows(lo, hi, n, seed):
    """Rows whose scale has an exponent in [lo, hi): half-way points of the codes and the floats next to them."""
    g = np.random.default_rng(seed)
    s = (np.ldexp(1 + g.random(n), g.integers(lo, hi, n))).astype(np.float32)
    x = (s[:, None].astype(np.float64) * (g.integers(-127, 127, (n, 64)) + 0.5)).astype(np.float32)
    x = np.where(g.random((n, 64)) < 0.3, np.nextafter(x, np.float32(np.inf)), x)
    x = np.where(g.random((n, 64)) < 0.3, np.nextafter(x, np.float32(-np.inf)), x)
    x[:, 0], x[:, 1] = -127 * s, 127 * s
    return x.astype(np.float32)


@pytest.mark.parametrize("lo,hi", [(-20, 20), (-104, -96), (96, 104), (-126, -100), (100, 120)])
def test_quantiser_codes_equal_ieee_division(lo, hi):
    import paper_2411_17178_amd as lv
    x = torch.from_numpy(_rows(lo, hi, 4001, lo + 1000))
    codes, sz = lv.litevar_qkv8_quantize(x.cuda())
    want_c, want_s, want_z = oracle.quantize_rows(workloads.to_oracle_array(x))
    sz = sz.cpu().numpy().astype(np.float64)
    assert np.array_equal(sz[:, 0], want_s) and np.array_equal(sz[:, 1], want_z)
    assert np.array_equal(codes.cpu().numpy().astype(np.int32), want_c)
