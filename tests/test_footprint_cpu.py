"""Admission estimates (host code only, no device needed)."""
import time

import numpy as np
import pytest

import inputs

pbm = pytest.importorskip("paper_2108_10481_amd")


def _lean(m, **kw):
    """The estimate without any workspace of the symmetric split."""
    if kw.get("precision", pbm.PB_FP64) == pbm.PB_FP32:
        kw["far_symmetric"] = -1
    else:
        kw["operator_mode"] = pbm.PB_AUTO
    return pbm.pb_estimate_device_bytes(m.xyz, m.tri, pbm.pb_default_options(**kw))


@pytest.mark.parametrize("freq", [2, 6, 10, 13])
@pytest.mark.parametrize("kw", [dict(), dict(precision=pbm.PB_FP32), dict(precision=pbm.PB_FP32, far_symmetric=1),
                                dict(source_chunks=1), dict(precision=pbm.PB_FP32, source_chunks=1)])
def test_server_takes_small_requests_without_room_for_the_split(freq, kw):
    """A request that fits without the symmetric split's slots is taken: the split
    (or, where it is asked for, the parts of its items) is left out."""
    m, shape = inputs.star_surface(4, freq, 5.0)
    c = inputs.charges_in_star(6, 3, shape)
    lean = _lean(m, **kw)
    if kw.get("far_symmetric") == 1:   # whole items: 2 slots of 64 bytes per triangle and range of 64
        chunks = max(m.n_triangles // 32, 1)
        ranges = -(-m.n_triangles // 64)
        lean += int(1.1 * 64 * m.n_triangles * max(0, 2 * ranges - 2 * chunks)) + 1
    with pbm.Server(hbm_budget=lean, max_slots=1) as s:
        t = s.submit(m.xyz, m.tri, c.xyz, c.q, pbm.pb_default_options(**kw))
        try:
            s.wait(t)
        except pbm.PbError as e2:      # no device here: only the admission is looked at
            assert e2.code == pbm.PB_E_DEVICE


def test_estimates_are_arithmetic():
    """2000 estimates of a large mesh: microseconds each, no work list is built."""
    xyz, tri = np.zeros((1000002, 3)), np.zeros((2000000, 3), dtype=np.int32)
    opt = pbm.pb_default_options(precision=pbm.PB_FP32)
    t0 = time.perf_counter()
    for _ in range(2000):
        pbm.pb_estimate_device_bytes(xyz, tri, opt)
    assert time.perf_counter() - t0 < 0.5
