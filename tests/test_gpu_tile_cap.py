"""GPU: the prediction's iteration cap where one work-group iterates on the residual
recursion.  The cap counts the updates up to the one that meets the stopping test, so a
cap of exactly the count that an uncapped solve reports is enough and gives its state to
the bit; one update less is not enough, and says so.
"""
import numpy as np
import pytest

from paper_1811_05579_amd import GrteBatch
from paper_1811_05579_amd.workloads import random_state

from test_gpu_parity import _ctx

pytestmark = pytest.mark.gpu

TOL = 1e-15


def _slab(N, nv, m, eps, cap):
    w = random_state(N, nv, seed=400 + N, m=m, eps=eps)
    g = _ctx(w)
    g.set_state(w.E, w.O, w.T)
    g.set_solver(TOL, cap, 100)
    info = g.step(0.5 / N, eps, info=True)
    out = info, g.get_state(), g.pred_history()
    g.close()
    return out


@pytest.mark.parametrize("N,nv,m,eps", [(100, 16, 3, 1e-2), (257, 32, 0, 1e-3), (512, 64, 3, 1e-1)])
def test_cap_of_a_slab(N, nv, m, eps):
    ref, state, hist = _slab(N, nv, m, eps, 200)
    n = ref["pred_iters"]
    assert ref["status"] == 0 and ref["pred_converged"] == 1 and n > 3 and hist.size == n
    info, same, h = _slab(N, nv, m, eps, n)
    assert info["status"] == 0 and info["pred_converged"] == 1 and info["pred_iters"] == n
    assert np.array_equal(h, hist)
    for a, b in zip(state, same):
        assert np.array_equal(a, b)
    info, _, h = _slab(N, nv, m, eps, n - 1)
    assert info["status"] == -4 and info["pred_converged"] == 0 and info["pred_iters"] == n - 1
    assert np.array_equal(h, hist[:n - 1])


def test_cap_of_the_reference_scheme():
    """Each Picard sweep's solve within the largest count that the sweeps report."""
    w = random_state(200, 16, seed=420, m=3, eps=0.5)
    got = []
    for cap in (200, None):
        g = _ctx(w)
        g.set_state(w.E, w.O, w.T)
        g.set_solver(TOL, cap or got[0][0]["pred_max_iters"], 100)
        got.append((g.reference_step(0.5 / w.N, w.eps), g.get_state()))
        g.close()
    assert got[0][0] == got[1][0] and got[0][0]["status"] == 0
    for a, b in zip(got[0][1], got[1][1]):
        assert np.array_equal(a, b)


def test_cap_of_a_batch():
    ws = [random_state(N, nv, seed=440 + N, m=m, eps=eps)
          for N, nv, m, eps in ((70, 8, 3, 1e-2), (300, 16, 0, 1e-3), (1100, 32, 3, 1e-2))]
    for w in ws:
        w.dt = 0.5 / w.N

    def run(cap):
        b = GrteBatch(ws)
        b.set_opacity(np.concatenate([w.sigma0 for w in ws]))
        b.set_inflow(np.concatenate([w.bL for w in ws]), np.concatenate([w.bR for w in ws]))
        b.set_state(*(np.concatenate([getattr(w, k).reshape(-1) for w in ws]) for k in ("E", "O", "T")))
        b.set_solver(TOL, cap, 100)
        out = (*b.step(info=True), b.get_state())
        b.close()
        return out

    status, ref, state = run(200)
    its = [i["pred_iters"] for i in ref]
    assert status == 0
    status, info, same = run(max(its))
    assert status == 0 and [i["pred_iters"] for i in info] == its
    for a, b in zip(state, same):
        assert np.array_equal(a, b)
    status, info, _ = run(max(its) - 1)
    assert status == -4
    assert [bool(i["pred_converged"]) for i in info] == [k < max(its) for k in its]
