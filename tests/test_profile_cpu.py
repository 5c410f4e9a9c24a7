"""What a profiled inference reports of the rows where some launches are a layer each and others several (csrc/spdnn_profile.h),
run through its host build: counts that the host was told go to their own layers, and nothing is written beyond the last."""
import ctypes

import numpy as np
import pytest

from paper_2007_14152_amd import build as hip_build


@pytest.mark.parametrize("L,runs,told", [
    (1, [(0, 1, 0)], []),                              # one layer, in a launch that keeps rows on the chip
    (2, [(0, 2, 0)], []),
    (6, [(0, 1, 1), (1, 2, 1), (2, 6, 0)], [1, 2]),     # the first two one by one
    (70, [(0, 2, 0), (2, 70, 0)], []),
])
def test_counts_of_launches(L, runs, told):
    lib = ctypes.CDLL(hip_build.ORDER_HOST_LIB)
    host = np.arange(1000, 1000 + L + 2, dtype=np.int32)
    rows = np.arange(L + 1 + 8, dtype=np.int32)        # L + 1 counters, and what lies behind them
    want = rows.copy()
    want[told] = host[told]
    flat = np.array(runs, dtype=np.int32)
    lib.spdnn_take_host_counts_host(flat.ctypes.data_as(ctypes.c_void_p), len(runs), host.ctypes.data_as(ctypes.c_void_p),
                                    rows.ctypes.data_as(ctypes.c_void_p))
    assert np.array_equal(rows, want)
