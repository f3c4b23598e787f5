"""GPU: exact neighbour sets at r_list where forces alone would not show a
lost pair: open and mixed axes with ghost rows, a batch of which some systems
were rebuilt, and rows longer than the general build keeps in LDS."""
import numpy as np
import pytest

from paper_1412_3387_amd import inputs
from tests.gpu_helpers import min_image_diff, neighbor_sets_equal

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1412_3387_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("periodic", [(0, 0, 0), (1, 0, 1), (0, 1, 0), (0, 0, 1)])
@pytest.mark.parametrize("order", ["sorted", "shuffled"])
@pytest.mark.parametrize("kind", ["lj_fp64", "lj_mixed", "dpd_fp64", "dpd_mixed"])
def test_open_frames_with_ghosts(orc, B, periodic, order, kind):
    """A frame whose open axes start at an offset, locals in its middle and
    ghosts around them up to its faces."""
    import torch
    rng = np.random.default_rng(501)
    if kind.startswith("lj"):
        density, r_cut, r_buff, kw = 0.8, 2.5, 0.4, dict(nlist_cap=176)
    else:
        density, r_cut, r_buff, kw = 3.0, 1.0, 0.5, dict(pair=B.PAIR_DPD, nlist_cap=104)
    L = np.array([17.3, 18.1, 16.6]) if kind.startswith("lj") else np.array([10.3, 11.1, 9.6])
    per = np.array(periodic)
    lo = np.where(per == 1, 0.0, np.array([-3.7, 2.9, -11.0]))
    n = int(density * np.prod(L))
    pos = lo + rng.uniform(0.0, 1.0, (n, 3)) * L
    pos[0], pos[1] = lo, lo + np.nextafter(1.0, 0.0) * L  # corners of the frame
    inner = np.all((per == 1) | ((pos >= lo + 0.18 * L) & (pos < lo + 0.82 * L)), axis=1)
    inner[:2] = False
    pos = np.concatenate([pos[inner], pos[~inner]])
    m = int(inner.sum())
    perm = np.concatenate([rng.permutation(m), np.arange(m, n)])  # shuffled rows, if unsorted
    tags = np.empty(n, dtype=np.int32)
    tags[:] = perm if order == "shuffled" else np.arange(n)
    ctx = B.Context([B.ModelParams(precision=B.FP64 if kind.endswith("fp64") else B.MIXED, r_cut=r_cut, r_buff=r_buff,
                                   sort_period=100 if order == "sorted" else 0, halo_cap=4096, **kw)],
                    [dict(pos=pos[tags[:m]], vel=np.zeros((m, 3)), tag=tags[:m], L=L, lo=lo, periodic=periodic,
                          n_cap=n + 70)])
    ctx.build_nlist(True)  # (Morton order, while there are no ghosts)
    rec = np.zeros(n - m, dtype=[("x", "f8", 3), ("v", "f8", 3 * kind.startswith("dpd")), ("tag", "i4"), ("pad", "i4")])
    rec["x"], rec["tag"] = pos[m:], np.arange(m, n)
    fields = B.FIELD_POS | B.FIELD_TAG | (B.FIELD_VEL if kind.startswith("dpd") else 0)
    ctx.unpack_ghosts(0, torch.as_tensor(rec.view(np.uint8).reshape(-1).copy(), device=ctx.device), n - m, fields,
                      B.GHOST_SELECT, np.where(per == 1, L, 1000.0))
    ctx.build_nlist(True)
    ctx.check()
    tag = ctx.tag[:n].cpu().numpy()
    x = ctx.pos[:n, :3].cpu().numpy()
    assert np.array_equal(x[np.argsort(tag)], pos)
    nn, rows = ctx.neighbor_rows(0)
    off, ref = orc.neighbors(pos, L, r_cut, r_buff, which=np.arange(m), periodic=periodic)
    for r in range(m):
        t = tag[r]
        assert np.array_equal(np.sort(tag[rows[r]]), ref[off[t]:off[t + 1]]), (r, int(t))


@pytest.mark.parametrize("sort", [100, 0])
@pytest.mark.parametrize("moved", [(1,), (0, 3), (4,), (0, 1, 2, 3, 4)])
def test_lists_of_a_batch_after_some_rebuilds(orc, B, sort, moved):
    """Five systems, of which some have a particle that moved past r_buff / 2:
    these have the lists of their new positions, the others keep those of
    their last build (framed and general tiles in all of them)."""
    rng = np.random.default_rng(502)
    sizes = (4000, 1037, 64, 6001, 130)
    sysd = []
    for k, n in enumerate(sizes):
        s = inputs.lj_fluid(n, 510 + k, 520 + k, density=0.8442 if n > 200 else 0.2)
        p = rng.permutation(n) if k % 2 else np.arange(n)  # every other one in random order
        sysd.append(dict(pos=s.pos[p], vel=s.vel[p], tag=p.astype(np.int32), L=s.L))
    ctx = B.Context([B.ModelParams(precision=B.FP64, sort_period=sort, halo_cap=6400)] * len(sizes), sysd)
    ctx.build_nlist(True)
    ctx.check()
    at_build = []
    for k, n in enumerate(sizes):
        o = ctx.offsets[k]
        tag = ctx.tag[o:o + n].cpu().numpy()
        x = ctx.pos[o:o + n, :3].cpu().numpy()[np.argsort(tag)]
        assert neighbor_sets_equal(orc, ctx, x, sysd[k]["L"], 2.5, 0.4, sys=k) == []
        at_build.append(x)
    for k in range(len(sizes)):
        # everyone moves a little (0.05 per axis at most: |d| < 0.09 < r_buff / 2),
        # and in the chosen systems one particle far
        n, o, L = sizes[k], ctx.offsets[k], sysd[k]["L"]
        x = ctx.pos[o:o + n, :3].cpu().numpy()
        x = x + rng.uniform(-0.05, 0.05, x.shape)
        if k in moved:
            x[rng.integers(n)] += np.array([0.3, -0.2, 0.1])
        ctx.pos[o:o + n, :3] = ctx.torch.as_tensor(inputs.wrap(x, L), device=ctx.device)
    before = ctx.build_count()
    ctx.build_nlist(False)
    ctx.check()
    assert ctx.build_count() == before + 1
    for k, n in enumerate(sizes):
        o = ctx.offsets[k]
        tag = ctx.tag[o:o + n].cpu().numpy()
        x = ctx.pos[o:o + n, :3].cpu().numpy()[np.argsort(tag)]
        assert np.max(np.abs(min_image_diff(x, at_build[k], sysd[k]["L"]))) < 0.4
        want = x if k in moved else at_build[k]
        assert neighbor_sets_equal(orc, ctx, want, sysd[k]["L"], 2.5, 0.4, sys=k) == []


@pytest.mark.parametrize("kind", ["lj_fp64", "lj_mixed", "dpd_mixed", "bonded"])
@pytest.mark.parametrize("block", [256, 512])
def test_long_rows_of_scattered_tiles(orc, B, kind, block):
    """Rows of 64 to 250 entries in random order: the general build keeps the
    first 128 of a row in LDS and the others in memory until they are
    numbered."""
    rng = np.random.default_rng(503)
    n, L = 2701, np.array([14.0, 15.0, 13.0])
    r_cut, r_buff, kw = 3.0, 0.4, dict()
    if kind == "dpd_mixed":
        kw = dict(pair=B.PAIR_DPD)
    if kind == "bonded":
        kw = dict(bond_cap=2, fene_R0=400.0)
    # twice as dense in one half of the box as in the other
    u = rng.uniform(0.0, 1.0, (n, 3))
    u[:, 0] = np.where(rng.uniform(size=n) < 2.0 / 3.0, 0.5 * u[:, 0], 0.5 + 0.5 * u[:, 0])
    pos = inputs.wrap(u * L, L)
    sysd = dict(pos=pos, vel=np.zeros_like(pos), L=L)
    bkw = {}
    if kind == "bonded":
        sysd["bonds"] = bkw["bonds"] = np.stack([np.arange(0, n - 1, 2), np.arange(1, n, 2)], axis=1).astype(np.int32)
    ctx = B.Context([B.ModelParams(precision=B.FP64 if kind in ("lj_fp64", "bonded") else B.MIXED, r_cut=r_cut,
                                   r_buff=r_buff, sort_period=0, nlist_cap=320, cell_cap=128, block_nlist=block, **kw)],
                    [sysd])
    ctx.build_nlist(True)
    ctx.check()
    nn, rows = ctx.neighbor_rows(0)
    assert ctx.general_tiles() == -(-n // 64)
    assert nn.min() < 128 < nn.max() and (nn > 128).sum() > 500
    assert neighbor_sets_equal(orc, ctx, pos, L, r_cut, r_buff, **bkw) == []
