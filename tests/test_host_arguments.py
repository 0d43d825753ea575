"""The two ways host arguments take into a call -- packed for one call, numpy arrays for a frozen one -- hold the same bytes and refuse the same."""
import warnings

import numpy as np
import pytest

from paper_2603_21365_amd import tide_route as tr

INF, NAN = float("inf"), float("nan")
FLOATS = [0.5, 1, True, [0.1, -0.0, INF], (1, 2.5, 16777217), [NAN, 1e-46, 3.4e38], [1e39, 0, 0], np.float64(0.1), np.arange(3.0), [np.float32(0.1)] * 3, [[0.1], [0.2]], [2.0], "x", [0.1, 0.2], [None] * 3, [True, False, 2]]
INTS = [3, -1, True, [3, 7, 11], (0, -2147483648, 2147483647), [3.7, 2.0, -1.5], 2.5, np.arange(3), [np.int64(4)] * 3, [2147483648, 0, 0], 1 << 40, [5], "x", [1, 2], [None] * 3]


def bytes_of(host, value, dtype):
    try:
        with warnings.catch_warnings():
            warnings.simplefilter("ignore")
            keep = host(value, 3, dtype)[0]
    except Exception as e:                          # noqa: BLE001 -- the kind of refusal is what is compared
        return type(e)
    return keep if isinstance(keep, bytes) else (keep.tobytes() if keep.dtype == dtype and keep.shape == (3,) else None)


@pytest.mark.parametrize("dtype,value", [(np.float32, v) for v in FLOATS] + [(np.int32, v) for v in INTS])
def test_one_call_and_frozen_call_agree(dtype, value):
    got, want = bytes_of(tr._host_once, value, dtype), bytes_of(tr._host, value, dtype)
    assert got == want and got is not None
