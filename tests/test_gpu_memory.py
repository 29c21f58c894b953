"""GPU: device memory of a slab's context.  The state (E and O, in and out), the stages E*
and O*, the right-hand sides and one buffer of partial sums are eight words per cell and
pair; only slabs whose sums every work-group forms itself have a second such buffer.
"""
import gc

import pytest

torch = pytest.importorskip("torch")

from paper_1811_05579_amd import Grte, gauss_legendre

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nv", [(4000, 120), (3900, 128)])
def test_words_per_cell_and_pair(N, nv):
    """Nine words bound the eight, the per-cell arrays and the padding to the solvers' rows
    and to the allocator's granules."""
    mu, om = gauss_legendre(nv)
    gc.collect()                                   # nothing of an earlier test is freed in between
    first = Grte(N, mu, om)                        # what the first context costs the process
    free = torch.cuda.mem_get_info()[0]
    gs = [Grte(N, mu, om) for _ in range(16)]
    used = free - torch.cuda.mem_get_info()[0]
    for g in gs + [first]:
        g.close()
    assert 0 < used <= 16 * 9 * 8 * N * (nv // 2)
