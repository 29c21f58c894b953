"""GPU: one slab's prediction where its form changes -- one work-group up to 512 cells and
32 pairs (two, four, six or eight rows per lane), else a work-group per pair (two to
sixteen rows per thread, the angular sum by every work-group up to 32 words per thread) --
against the oracle at the parity bars; and a group of slabs of both sizes.
"""
import numpy as np
import pytest

from paper_1811_05579_amd import step_group
from paper_1811_05579_amd.workloads import random_state

from test_gpu_parity import _ctx, compare

pytestmark = pytest.mark.gpu

# (N, nv, m, eps)
EDGES = [(2, 2, 0, 1.0), (3, 64, 3, 1e-2), (64, 16, 3, 1e-3), (128, 18, 0, 1e-2), (129, 2, 3, 1e-4), (256, 8, 0, 1e-3),
         (257, 32, 3, 1e-2), (384, 6, 0, 1.0), (385, 14, 3, 1e-3), (512, 64, 0, 1e-2),
         (100, 66, 3, 1e-2), (512, 66, 0, 1e-3), (513, 16, 3, 1e-2), (513, 18, 0, 1e-2), (1024, 8, 3, 1e-3),
         (1025, 8, 0, 1e-2), (2048, 10, 3, 1e-2), (2049, 4, 0, 1e-3), (4096, 2, 3, 1e-2)]


@pytest.mark.parametrize("N,nv,m,eps", EDGES)
def test_prediction_form_edges(N, nv, m, eps):
    w = random_state(N, nv, seed=900 + N + nv, m=m, eps=eps)
    w.dt = 0.5 / N
    compare(w, w.E, w.O, w.T)


@pytest.mark.parametrize("shapes", [[(100, 8), (512, 66), (300, 4)], [(130, 16), (512, 6), (2, 2)]])
def test_group_of_both_forms(shapes):
    """Every slab of a group takes the form that it takes alone: its state is that of its own step, to the bit."""
    ws = [random_state(N, nv, seed=950 + N, m=0, eps=1e-2) for N, nv in shapes]
    gs = [_ctx(w) for w in ws]
    for g, w in zip(gs, ws):
        g.set_state(w.E, w.O, w.T)
    step_group(gs, [0.5 / w.N for w in ws], [w.eps for w in ws])
    for g, w in zip(gs, ws):
        one = _ctx(w)
        one.set_state(w.E, w.O, w.T)
        one.step(0.5 / w.N, w.eps)
        for a, b in zip(g.get_state(), one.get_state()):
            assert np.array_equal(a, b)
        one.close()
        g.close()


# work-groups of eight wavefronts (more than 2048 cells): ragged ends, pairs that the two
# lanes of a position do not share evenly, more pairs than one batch of sums
@pytest.mark.parametrize("N,nv,m,eps", [(2050, 10, 3, 1e-4), (3001, 22, 0, 1e-2), (4095, 36, 3, 1e-3)])
def test_wide_work_group(N, nv, m, eps):
    w = random_state(N, nv, seed=970 + N, m=m, eps=eps)
    w.dt = 0.5 / N
    compare(w, w.E, w.O, w.T)
