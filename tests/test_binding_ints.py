"""How the binding lays host ints out for the library: the fast conversion and the general one behind it."""
import ctypes

import numpy as np
import pytest

from paper_2407_00079_amd import binding as B


def read(ints, code, n):
    return list(((ctypes.c_int32 if code == "i" else ctypes.c_int64) * n).from_address(ints.at))


@pytest.mark.parametrize("code", ["i", "q"])
@pytest.mark.parametrize("values", [[3, 0, 7], (5,), np.array([1, 2 ** 30]), [2.0, 3.9], [np.int64(4), 5], range(65)])
def test_values_arrive(code, values):
    n = len(values)
    assert read(B._Ints(code, values, n), code, n) == [int(x) for x in values]


def test_short_empty_long_and_wide():
    assert read(B._Ints("i", [9], 3), "i", 3) == [9, 0, 0]          # the missing entries are zero, and there
    assert B._Ints("q", [], 0).at != 0
    assert read(B._Ints("i", [2 ** 32 + 5], 1), "i", 1) == [5]      # what ctypes makes of it
    with pytest.raises(IndexError):
        B._Ints("i", [1, 2, 3], 2)
