"""GPU: liquids that fill part of their box, flat boxes and long cut-offs.  The
capacities, not the mean density, say how many members a tile's plan has to
hold and how many halo entries the force pass stages: the tiles of a droplet
take the framed build and the common pair loop; so do those of a flat box or a
long cut-off.  Lists and forces are the oracle's."""
import numpy as np
import pytest

from paper_1412_3387_amd import inputs
from tests.gpu_helpers import frel, neighbor_sets_equal

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


def flat_liquid():
    """A jittered simple cubic liquid of 90 x 90 x 18.5, 18 layers: its tiles
    are as flat as the box."""
    a, m, k = 1.06, 85, 18
    g = np.arange(m) * a
    z = np.arange(k) * (18.5 / k)
    p = np.stack(np.meshgrid(g, g, z, indexing="ij"), axis=-1).reshape(-1, 3)
    L = np.array([m * a, m * a, 18.5])
    rng = np.random.default_rng(311)
    pos = inputs.wrap(p + 0.25 + rng.uniform(-0.05, 0.05, p.shape), L)
    return pos, inputs.maxwell_velocities(len(pos), 1.0, 312), L


@pytest.mark.parametrize("what", ["droplet", "slab", "flat", "long"])
def test_few_tiles_reach_beyond_the_stage(orc, B, what):
    """At most one tile in ten takes the slower pair loop, and the forces of
    both loops are the oracle's."""
    kw, r_cut, r_buff = dict(CAPS), 2.5, 0.4
    if what == "droplet":
        pos, vel, L = part_of_box(32000, (3, 3, 3))
    elif what == "slab":
        pos, vel, L = part_of_box(32000, (1, 1, 3))
    elif what == "flat":
        pos, vel, L = flat_liquid()
        kw, r_buff = dict(), 0.9
    else:
        s = inputs.lj_fluid(32000, 301, 302)
        pos, vel, L = s.pos, s.vel, s.L
        kw, r_cut = dict(nlist_cap=440), 4.0
    ctx = B.Context([B.ModelParams(precision=B.FP64, r_cut=r_cut, r_buff=r_buff, sort_period=100, **kw)],
                    [dict(pos=pos, vel=vel, L=L)])
    ctx.build_nlist(True)
    ctx.compute_forces(0, 0)
    ctx.check()
    assert ctx.rare_tiles() <= -(-len(pos) // 64) // 10
    which = np.sort(np.random.default_rng(6).choice(len(pos), 300, replace=False))
    x, v, f, tag = ctx.host_state()
    F = orc.pair_forces("lj", pos, L, [1.0, 1.0, r_cut], which=which)[0]
    assert frel(f[np.argsort(tag)][which, :3], F) <= 1e-12
