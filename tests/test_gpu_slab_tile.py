"""The tile that solves a slab's prediction (factor once, one right-hand side per
update) at the sizes where its row layout changes: 64 lanes of M = 4, 6, .. 32 rows,
so one cell below, at and above a multiple of 128; the smallest and the largest slab;
fewer pairs than wavefronts, as many, and one more.  Against the oracle's step at the
FP64 bar of the batched parity tests (fp64_bar.py): 1e-12 up to a stiffness of 1e6,
ten times the oracle's own one-ulp sensitivity above it."""
import numpy as np
import pytest

from fp64_bar import FLOOR, STIFF, bars, sensitivity, stiffness
from oracle.ap1d import Physics, ap_step
from paper_1811_05579_amd import GrteBatch
from paper_1811_05579_amd.workloads import Ensemble, random_state

pytestmark = pytest.mark.gpu
KEYS = ("T", "E", "O")

# (N, nv, m, eps)
EDGES = [(2, 2, 3, 1e-2), (3, 32, 0, 1.0), (127, 16, 3, 1e-3), (128, 18, 0, 1e-2), (129, 4, 3, 1e-4),
         (255, 8, 0, 1e-3), (383, 4, 3, 1e-2), (384, 6, 0, 1e-4), (385, 4, 3, 1.0), (641, 4, 0, 1e-2),
         (1024, 4, 3, 1e-3), (1025, 2, 0, 1e-2), (1153, 2, 3, 1e-1), (1663, 2, 0, 1e-3), (1793, 2, 3, 1e-2),
         (2047, 2, 0, 1e-2), (2048, 2, 3, 1e-4)]


@pytest.mark.parametrize("wave_max_n", [0, 256])
def test_tile_edges(wave_max_n):
    ms = []
    for q, (N, nv, m, eps) in enumerate(EDGES):
        w = random_state(N, nv, seed=700 + q, m=m, eps=eps)
        w.dt = 0.5 / N
        ms.append(w)
    pk = Ensemble("edges", ms).packed()
    b = GrteBatch(ms)
    b.set_tuning(wave_max_n, b.get_tuning()["grid"])
    b.set_opacity(pk["sigma0"])
    b.set_inflow(pk["bL"], pk["bR"])
    b.set_state(pk["E"], pk["O"], pk["T"])
    st, infos = b.step(info=True)
    assert st == 0, infos
    for w, got in zip(ms, b.split(*b.get_state())):
        step = lambda E, O, T, s: ap_step(E, O, T, s, w.mu, w.omega, w.bL, w.bR,
                                          Physics(a=w.a, c=w.c, Cv=w.Cv, eps=w.eps, dt=w.dt, L=w.L, m=w.m))
        if stiffness(w, w.T) <= STIFF:
            ref, bar = step(w.E, w.O, w.T, w.sigma0), {k: FLOOR for k in KEYS}
        else:
            ref, sens = sensitivity(step, [w.E, w.O, w.T, w.sigma0], KEYS)
            bar = bars(w, w.T, KEYS, sens)
        for name, x in zip(("E", "O", "T"), got):
            err = np.max(np.abs(x - ref[name])) / np.max(np.abs(ref[name]))
            assert err <= bar[name], (w.name, name, err, bar[name])
    b.close()
