"""GPU: the diffusion step where its work-group changes shape -- one wavefront's last
row, four wavefronts full, sixteen with one, two and four cells per thread -- against
the oracle at the bar of the one-step test (1e-12 of the largest value).
"""
import pytest

from oracle.diffusion1d import three_stage_step
from paper_1811_05579_amd import GrteDiff

from test_gpu_diffusion import _rel, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [2, 63, 64, 65, 255, 258, 1023, 1024, 1025, 2047, 2049, 4095])
@pytest.mark.parametrize("m,bc,ck", [(0, "neumann", "old"), (3, "dirichlet", "predicted")])
def test_step_at_work_group_edges(N, m, bc, ck):
    T, sigma0 = _state(N, N + m)
    g = GrteDiff(N, opacity_law=m, boundary=bc, ghost=(1.0, 0.1))
    g.set_opacity(sigma0)
    g.set_state(T)
    info = g.step(0.5 / N, corr_K=ck, info=True)
    assert info["status"] == 0
    Tg, Ug = g.get_state()
    To, Uo = three_stage_step(T, sigma0, 0.5 / N, m=m, bc=bc, ghost_T=(1.0, 0.1), corr_K=ck)
    assert _rel(Ug, Uo) <= 1e-12
    assert _rel(Tg, To) <= 1e-12
    g.close()
