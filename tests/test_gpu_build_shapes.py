"""GPU: the values that `tpp_nlist` takes are one list build, entry by entry."""
import numpy as np
import pytest

from paper_1412_3387_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1412_3387_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("block", [512, 256])
@pytest.mark.parametrize("kind", ["lj", "melt", "dpd"])
def test_one_build_for_every_tpp_nlist(B, kind, block):
    if kind == "lj":
        s, kw = inputs.lj_fluid(20000, 401, 402), dict(precision=B.MIXED)
    elif kind == "melt":
        s, kw = inputs.polymer_melt(200, 403), dict(precision=B.FP64, pair=B.PAIR_WCA, bond_cap=2)
    else:
        s, kw = inputs.dpd_fluid(20000, 404, 405), dict(precision=B.MIXED, pair=B.PAIR_DPD, r_cut=1.0, r_buff=0.5)
    got = []
    for w in (64, 32):
        ctx = B.Context([B.ModelParams(sort_period=100, tpp_nlist=w, block_nlist=block, **kw)],
                        [dict(pos=s.pos, vel=s.vel, L=s.L, tag=s.tag, bonds=s.bonds)])
        ctx.build_nlist(True)
        ctx.check()
        nn, rows = ctx.neighbor_rows(0)
        got.append((nn, np.concatenate([np.asarray(r) for r in rows])))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
