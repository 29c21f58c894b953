"""GPU: the timing of the 2-D operator product counts products that ran.  A solve whose
start already meets the tolerance runs none, whatever the last solve took.
"""
import pytest

from paper_1811_05579_amd.workloads import random_state_2d

from test_gpu_ap2d import _ctx

pytestmark = pytest.mark.gpu


def test_accepted_start_times_no_product():
    w = random_state_2d(33, 21, 16, seed=31, m=3, eps=1e-1)
    g = _ctx(w)
    g.set_state(w.E, w.Ox, w.Oy, w.T)
    g.set_profiling(True)
    info = g.step(w.dt, w.eps, info=True)
    ms, n = g.read_timing()
    assert info["status"] == 0 and info["pred_iters"] > 0 and info["corr_iters"] > 0 and info["corr_narrow"] == 1
    assert n > 0 and ms > 0.0
    g.set_solver(1e6)
    g.set_profiling(True)
    info = g.step(w.dt, w.eps, info=True)
    assert info["pred_iters"] == 0 and info["corr_iters"] == 0
    assert g.read_timing() == (0.0, 0)
    g.close()
