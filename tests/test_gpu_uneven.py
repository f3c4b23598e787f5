"""GPU: liquids that fill part of their box.  The cells' capacity, not the
mean density, says how many members a tile's plan has to hold: the tiles of a
droplet or a slab take the framed build, and their lists are the oracle's."""
import numpy as np
import pytest

from paper_1412_3387_amd import inputs
from tests.gpu_helpers import neighbor_sets_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1412_3387_amd import binding
    binding.lib()
    return binding


def part_of_box(n, factors):
    """An LJ liquid in the middle of a box that is factors times longer."""
    s = inputs.lj_fluid(n, 301, 302)
    L = s.L * np.array(factors, dtype=np.float64)
    return s.pos + 0.5 * (L - s.L), s.vel, L


CAPS = dict(nlist_cap=152, cell_cap=56, halo_cap=4096)


@pytest.mark.parametrize("factors", [(3, 3, 3), (2, 2, 2), (1, 1, 3)])
@pytest.mark.parametrize("n", [4000, 32000])
def test_tiles_of_a_droplet_are_framed(orc, B, n, factors):
    pos, vel, L = part_of_box(n, factors)
    ctx = B.Context([B.ModelParams(precision=B.FP64, sort_period=100, **CAPS)], [dict(pos=pos, vel=vel, L=L)])
    ctx.build_nlist(True)
    ctx.check()
    # (a box of few cells, and a slab's short axes, may be too small for a tile's frame)
    if n == 32000 and min(factors) > 1:
        assert ctx.general_tiles() == 0
    which = np.sort(np.random.default_rng(5).choice(n, 400, replace=False))
    assert neighbor_sets_equal(orc, ctx, pos, L, 2.5, 0.4, which=which) == []
