"""Planning of the path pass (CPU): the layout choice and the work list of a
batch, through the library's host code.
"""
import ctypes
import os
import time

import pytest

from paper_2106_07927_amd import sgm

FAKE = 1 << 20


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(sgm.LIB_PATH):
        pytest.skip("libsgm.so not built")
    return sgm.load_library()


def workspace_seconds(lib, n):
    """Best of three sgm_batch_workspace_bytes calls over n small pairs of
    different sizes and one disparity range (the layout choice included)."""
    prm = sgm.SgmParams(9, 7, 8, 10, 120, 1, 1)
    pairs = (sgm.SgmPair * n)()
    for i in range(n):
        w, h = 100 + i % 211, 80 + i % 163
        pairs[i] = sgm.SgmPair(FAKE, FAKE, w, h, w, 64, FAKE, None)
    best = float("inf")
    for _ in range(3):
        t = time.perf_counter()
        assert lib.sgm_batch_workspace_bytes(pairs, n, ctypes.byref(prm), None) > 0
        best = min(best, time.perf_counter() - t)
    return best


def test_planning_time_grows_with_the_number_of_pairs(lib):
    """16 times the pairs take about 16 times as long (sorting adds little); a
    choice that looks at every pair for every pair would take 256 times."""
    assert workspace_seconds(lib, 4800) < 64 * max(workspace_seconds(lib, 300), 1e-4)
