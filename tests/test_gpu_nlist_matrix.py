"""GPU parity of the matrix build of the neighbour list at its edges: pairs at
r_list to the last bit (decided in FP64 beside the FP32 matrix results),
members that fill one, two and more passes, tiles of one row, bonded
exclusions on the same lattice."""
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


def _lattice(m, a, seed):
    """m^3 sites a apart, shifted as a whole: the separations a, 2a, ... come
    out in FP64 as either side of the exact multiple."""
    g = np.arange(m) * a
    z, y, x = np.meshgrid(g, g, g, indexing="ij")
    pos = np.stack([x.ravel(), y.ravel(), z.ravel()], axis=1)
    L = np.full(3, m * a)
    return inputs.wrap(pos + np.random.default_rng(seed).uniform(0, a, 3), L), L


# (sites per side, spacing, r_cut, r_buff): r_list = 2a, 3a or sqrt(2) a
@pytest.mark.parametrize("m,a,rc,rb", [(12, 1.45, 2.5, 0.4), (13, 0.9, 2.3, 0.4), (9, 2.05, 2.5, 2.05 * np.sqrt(2) - 2.5),
                                       (16, 0.62, 1.4, 0.46), (7, 1.45, 2.5, 0.4)])
def test_pairs_at_the_list_radius(orc, B, m, a, rc, rb):
    pos, L = _lattice(m, a, m)
    for sort in (1, 0):
        ctx = B.Context([B.ModelParams(precision=B.FP64, r_cut=rc, r_buff=rb, sort_period=sort, nlist_cap=160)],
                        [dict(pos=pos, vel=np.zeros_like(pos), L=L)])
        ctx.build_nlist(True)
        ctx.check()
        assert neighbor_sets_equal(orc, ctx, pos, L, rc, rb) == []


# 0.8442: most tiles in one pass; 2.2: 3,000 members near a tile, two passes and more
@pytest.mark.parametrize("n,density,shape", [(4033, 0.8442, (64, 256)), (6000, 2.2, (64, 256)), (6000, 2.2, (32, 512)),
                                             (6000, 2.2, (64, 512)), (2049, 0.3, (64, 256))])
def test_passes_and_remainders(orc, B, n, density, shape):
    s = inputs.lj_fluid(n, 71, 72, density=density)
    ctx = B.Context([B.ModelParams(precision=B.FP64, sort_period=1, tpp_nlist=shape[0], block_nlist=shape[1])],
                    [dict(pos=s.pos, vel=s.vel, L=s.L)])
    ctx.build_nlist(True)
    ctx.check()
    assert neighbor_sets_equal(orc, ctx, s.pos, s.L, 2.5, 0.4) == []
    # the halo lists each neighbour of the tile once
    nn, rows = ctx.neighbor_rows()
    for t, h in enumerate(ctx.halo_sizes()):
        assert h == len(np.unique(np.concatenate([r for r in rows[64 * t:64 * t + 64]] or [np.zeros(0)])))


@pytest.mark.parametrize("bond_cap", [2, 4])
def test_bonded_lattice_at_the_list_radius(orc, B, bond_cap):
    """Exclusions found through the tile's partner-tag table, partners in the
    same and in other tiles, on a lattice with pairs at r_list; tags shuffled."""
    m = inputs.polymer_melt(60, seed_vel=73)
    perm = np.random.default_rng(74).permutation(m.n)
    inv = np.argsort(perm)
    pos, bonds = m.pos[perm], inv[m.bonds]
    if bond_cap == 4:
        # every bead also bonded along the chain's next-nearest beads
        extra = [(c * 50 + k, c * 50 + k + 2) for c in range(60) for k in range(48)]
        bonds = np.concatenate([bonds, inv[np.array(extra)]])
    ctx = B.Context([B.ModelParams(precision=B.FP64, pair=B.PAIR_WCA, bond_cap=bond_cap, sort_period=1, fene_R0=9.0)],
                    [dict(pos=pos, vel=m.vel, L=m.L, bonds=bonds.astype(np.int32))])
    ctx.build_nlist(True)
    ctx.check()
    assert neighbor_sets_equal(orc, ctx, pos, m.L, 2.0 ** (1.0 / 6.0), 0.4, bonds=bonds.astype(np.int32)) == []


# boxes with more cells than the bitmap of stencil cells covers (131,072) and
# with fewer, two cells across an axis (nearest images), one row in the last tile
@pytest.mark.parametrize("n,L,shape", [(5000, (160.0, 161.0, 158.0), (64, 256)), (5000, (147.0, 147.0, 147.0), (64, 256)),
                                       (1985, (6.5, 30.0, 12.0), (64, 256)), (1985, (6.5, 30.0, 12.0), (32, 512)),
                                       (4097, (18.0, 18.0, 18.0), (64, 512)), (65, (9.0, 6.0, 6.0), (32, 256))])
@pytest.mark.parametrize("bonded", [False, True])
def test_scattered_rows_in_the_general_build(orc, B, n, L, shape, bonded):
    """Rows in random order: no tile fits one frame, every row reads its own
    stencil, in the same launch as the framed tiles."""
    rng = np.random.default_rng(n)
    L = np.array(L)
    pos = inputs.wrap(rng.uniform(0, 1, (n, 3)) * L, L)
    sysd = dict(pos=pos, vel=np.zeros_like(pos), L=L)
    bonds = None
    if bonded:
        bonds = sysd["bonds"] = np.stack([np.arange(0, n - 1, 2), np.arange(1, n, 2)], axis=1).astype(np.int32)
    ctx = B.Context([B.ModelParams(precision=B.FP64, sort_period=0, nlist_cap=256, tpp_nlist=shape[0],
                                   block_nlist=shape[1], bond_cap=2 if bonded else 0, fene_R0=400.0)], [sysd])
    ctx.build_nlist(True)
    ctx.check()
    assert ctx.general_tiles() > 0
    kw = dict(bonds=bonds) if bonded else {}
    assert neighbor_sets_equal(orc, ctx, pos, L, 2.5, 0.4, **kw) == []
