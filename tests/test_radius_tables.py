"""Radius tables as lists: the walk over the lists and the general path give the same descriptor, and both refuse the same."""
import ctypes as C

import numpy as np
import pytest

from paper_2411_17178_amd import binding


def _tables(H, K, value):
    return [[[value(h, k, j) for j in range(K)] for k in range(K)] for h in range(H)]


def _flat(rows, K):
    d = binding._make_desc((1,) * K, 1, rows, 0, None)
    return d.n_heads, list(C.cast(d.radius_per_head, C.POINTER(C.c_int32))[:len(rows) * K * K])


@pytest.mark.parametrize("H,K", [(1, 1), (3, 2), (30, 10), (2, 32)])
@pytest.mark.parametrize("form", ["list", "tuple", "bool", "numpy", "float", "array"])
def test_forms(H, K, form):
    rows = _tables(H, K, lambda h, k, j: (h * 7 + k * 3 + j) % 1025 - 1)
    want = [x for t in rows for r in t for x in r]
    if form == "tuple":
        rows = tuple(tuple(tuple(r) for r in t) for t in rows)
    elif form == "bool":
        rows, want = _tables(H, K, lambda h, k, j: (h + k + j) % 2 == 0), None
        want = [int(x) for t in rows for r in t for x in r]
    elif form == "numpy":
        rows = [[[np.int64(x) for x in r] for r in t] for t in rows]
    elif form == "float":
        rows = [[[x + 0.0 for x in r] for r in t] for t in rows]
    elif form == "array":
        rows = np.array(rows)
    assert _flat(rows, K) == (H, want)
    assert (binding._radius_tables(rows, K) is not None) == (form in ("list", "tuple")) or binding._tables_module is False


@pytest.mark.parametrize("rows", [[[[1, 2], [3, 4]], [[1, 2], [3]]], [[[1, 2], [3, 4]], [[1, 2]]],
                                  [[[1, 2, 3], [3, 4]]], [[[1, 2], [3, 4], [5, 6]]]])
def test_ragged_tables_are_refused(rows):
    with pytest.raises((AssertionError, TypeError)):
        binding._make_desc((1, 2), 1, rows, 0, None)


def test_values_beyond_the_type():
    for big in (2 ** 31, -2 ** 31 - 1, 2 ** 80):
        assert binding._radius_tables([[[big]]], 1) is None
    if binding._tables_module is False:
        pytest.skip("built without the interpreter's headers")
    assert bytes(binding._radius_tables([[[2 ** 31 - 1]], [[-2 ** 31]]], 1)) == np.array([2 ** 31 - 1, -2 ** 31], np.int32).tobytes()
