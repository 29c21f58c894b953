"""GPU: a group of small slabs that differ in the prediction's form (one work-group, or a
work-group per pair) or in rows per lane.  Every slab gets the bits of its own step, and the
predictions run beside each other, not one after the other.
"""
import numpy as np
import pytest

from paper_1811_05579_amd import step_group
from paper_1811_05579_amd.workloads import random_state

from test_gpu_parity import _ctx

pytestmark = pytest.mark.gpu

# (N, nv): two, four, six, eight rows per lane; both forms, the pairs' twice; both at their edges
GROUPS = [[(128, 16), (129, 2), (384, 10), (385, 64)],
          [(512, 66), (2, 2), (300, 128), (257, 64)],
          [(100, 66), (512, 64)]]


def _group(shapes, coop):
    ws = [random_state(N, nv, seed=1200 + N + nv, m=3, eps=(1e-2, 1e-3, 1.0)[i % 3]) for i, (N, nv) in enumerate(shapes)]
    gs = [_ctx(w) for w in ws]
    for g, w in zip(gs, ws):
        g.set_state(w.E, w.O, w.T)
        g.set_launch(cooperative=coop)
    return ws, gs, [0.5 / w.N for w in ws], [w.eps for w in ws]


@pytest.mark.parametrize("coop", [True, False])
@pytest.mark.parametrize("shapes", GROUPS)
def test_bits_of_the_single_steps(shapes, coop):
    ws, gs, dts, eps = _group(shapes, coop)
    _, ones, _, _ = _group(shapes, coop)
    for _ in range(4):
        infos = step_group(gs, dts, eps, info=True)
        for g, one, dt, e, i in zip(gs, ones, dts, eps, infos):
            ref = one.step(dt, e, info=True)
            assert ref["status"] == 0 and ref == i and i["sync_error"] == 0
            assert np.array_equal(g.pred_history(), one.pred_history())
            for a, b in zip(g.get_state(), one.get_state()):
                assert np.array_equal(a, b)
    for g in gs + ones:
        g.close()


@pytest.mark.parametrize("shapes", [[(128, 64), (256, 64), (384, 64), (512, 64)], [(512, 64), (512, 66)]])
def test_predictions_run_together(shapes):
    """The group's prediction takes well below the sum of its slabs' own."""
    ws, gs, dts, eps = _group(shapes, False)
    _, ones, _, _ = _group(shapes, False)

    def predict_ms(owner, step, n=50):
        for _ in range(5):
            step()
        owner.set_profiling(1)
        for _ in range(n):
            step()
        return owner.read_timing()["predict"][0] / n

    own = [predict_ms(o, lambda o=o, dt=dt, e=e: o.step(dt, e)) for o, dt, e in zip(ones, dts, eps)]
    together = predict_ms(gs[0], lambda: step_group(gs, dts, eps))
    assert together < max(own) + 0.6 * (sum(own) - max(own)), (together, own)
    for g in gs + ones:
        g.close()
