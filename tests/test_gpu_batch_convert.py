"""GPU: the batch's binary32 storage at the edges of its 128-cell blocks -- one cell less,
as many, one more; one pair and the most -- a round trip returns the stored values:
O rounded to binary32, E the binary64 sum of a c T^4 and the rounded deviation.
"""
import numpy as np
import pytest

from paper_1811_05579_amd import GrteBatch
from paper_1811_05579_amd.workloads import Ensemble, random_state

pytestmark = pytest.mark.gpu


def test_round_trip_at_block_edges():
    ms = [random_state(N, nv, seed=800 + N + nv, m=3, eps=1e-2)
          for N, nv in [(2, 2), (127, 6), (128, 128), (129, 16), (255, 2), (256, 64), (257, 10), (2048, 4)]]
    pk = Ensemble("edges", ms).packed()
    b = GrteBatch(ms)
    b.set_opacity(pk["sigma0"])
    b.set_inflow(pk["bL"], pk["bR"])
    b.set_storage(True)
    b.set_state(pk["E"], pk["O"], pk["T"])
    for w, (E, O, T) in zip(ms, b.split(*b.get_state())):
        base = (w.a * w.c * (w.T * w.T) * (w.T * w.T))[:, None]
        dev = (w.E - base).astype(np.float32)
        assert np.array_equal(T, w.T)
        assert np.array_equal(O, w.O.astype(np.float32).astype(np.float64))
        # the device may fuse a c T^4 into the difference and the sum: one rounding of the
        # large term (2^-53), one of the deviation (2^-24)
        assert np.all(np.abs(E - (base + dev.astype(np.float64))) <= 2.0 ** -52 * np.abs(base) + 2.0 ** -23 * np.abs(dev))
    b.close()
