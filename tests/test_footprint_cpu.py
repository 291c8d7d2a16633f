"""Admission estimates (host code only, no device needed)."""
import time

import numpy as np
import pytest

pbm = pytest.importorskip("paper_2108_10481_amd")


def test_estimates_are_arithmetic():
    """2000 estimates of a large mesh: microseconds each, no work list is built."""
    xyz, tri = np.zeros((1000002, 3)), np.zeros((2000000, 3), dtype=np.int32)
    opt = pbm.pb_default_options(precision=pbm.PB_FP32)
    t0 = time.perf_counter()
    for _ in range(2000):
        pbm.pb_estimate_device_bytes(xyz, tri, opt)
    assert time.perf_counter() - t0 < 0.5
