"""GPU: the values that `tpp_nlist` takes are one list build, entry by entry,
and the autotuner times each build once."""
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


@pytest.mark.parametrize("kind", ["lj", "dpd"])
def test_autotune_times_a_build_once(B, kind):
    """The two values of tpp_nlist report the time of their one build, and the
    first of them is the one chosen."""
    s = inputs.lj_fluid(20000, 411, 412) if kind == "lj" else inputs.dpd_fluid(20000, 413, 414)
    kw = dict() if kind == "lj" else dict(pair=B.PAIR_DPD, r_cut=1.0, r_buff=0.5)
    ctx = B.Context([B.ModelParams(precision=B.MIXED, sort_period=100, **kw)],
                    [dict(pos=s.pos, vel=s.vel, L=s.L, tag=s.tag)])
    t = ctx.autotune(1)
    ctx.check()
    bm = list(t.build_ms)
    assert min(bm) > 0 and bm[2:] == bm[:2]
    assert (t.tpp_nlist, t.block_nlist) == (64, 512 if bm[0] <= bm[1] else 256)
