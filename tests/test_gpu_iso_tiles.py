"""GPU: the tiled isotropic correction at the edges of its regions.

A region is 64 cells across and a multiple of 16 down; it takes no halo on a side it
covers, all steps in one launch (24 at most) if that holds for both, else nine per launch.
The per-step launches give the same map to the bit.
"""
import numpy as np
import pytest

from paper_1811_05579_amd.workloads import random_state_2d

from test_gpu_ap2d import _ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,steps", [(64, 96, 26), (65, 96, 19), (64, 97, 19), (63, 17, 25), (47, 33, 19),
                                         (93, 31, 12), (2, 130, 19), (130, 2, 19)])
def test_tiles_equal_per_step(nx, ny, steps):
    w = random_state_2d(nx, ny, 8, 300 + steps + nx, m=0, eps=1e-3, sigma=(1.0, 100.0))
    out = []
    for kind in ("chebyshev", "chebyshev-per-step"):
        g = _ctx(w)
        g.set_isotropic_correction(kind, steps)
        g.set_state(w.E, w.Ox, w.Oy, w.T)
        info = g.step(w.dt, w.eps, info=True)
        assert info["status"] == 0, info
        out.append((g.get_state(), info["pred_iters"]))
        g.close()
    assert out[0][1] == out[1][1]
    for a, b in zip(out[0][0], out[1][0]):
        assert np.array_equal(a, b)
