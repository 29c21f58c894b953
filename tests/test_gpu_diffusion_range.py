"""GPU: the diffusion schemes without a Newton solve at the end of the number range.  A heat
capacity of the radiation 4 a_t T^3 that overflows leaves U* = T^4, and the two-stage
scheme's T with it (the other's T gets a_t times the rounding of U* - T^4).
"""
import numpy as np
import pytest

from paper_1811_05579_amd import GrteDiff

from test_gpu_diffusion import _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", [1, 2])
@pytest.mark.parametrize("N", [37, 300, 1500, 3000])
def test_infinite_heat_capacity(N, scheme):
    T, sigma0 = _state(N, N)
    T = T + 2.0                                      # 4e308 T^3 overflows, T^4 does not
    g = GrteDiff(N, opacity_law=3, boundary="dirichlet", ghost=(1.0, 0.1))
    g.set_opacity(sigma0)
    g.set_state(T)
    assert g.step(0.5 / N, scheme=scheme, a_time=1e308, info=True)["status"] == 0
    Tg, Ug = g.get_state()
    g.close()
    assert np.max(np.abs(Ug - T ** 4) / T ** 4) <= 1e-15
    if scheme == 1:
        assert np.max(np.abs(Tg - T) / T) <= 1e-15
