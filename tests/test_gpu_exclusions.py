"""Bonded exclusions where a partner's tag is near a tile many times (ghost
copies of a partner that reach a small frame from several sides): no copy may
stay in the partner's row."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1412_3387_amd import binding
    binding.lib()
    return binding


# a wave keeps eight staged places per row: as many copies, one fewer and one
# more, and most of a cell
@pytest.mark.parametrize("block", [256, 512])
@pytest.mark.parametrize("copies", [1, 7, 8, 9, 60])
@pytest.mark.parametrize("bond_cap", [1, 4])
def test_every_copy_of_a_partner_is_excluded(B, copies, bond_cap, block):
    import torch
    rng = np.random.default_rng(copies)
    L, n, rl = np.full(3, 12.0), 64, 2.9
    pos = 5.0 + 2.0 * rng.uniform(size=(n, 3))
    pairs = [(0, 1), (2, 3)] + ([(0, 5), (0, 6), (0, 7)] if bond_cap == 4 else [])
    ctx = B.Context([B.ModelParams(precision=B.FP64, bond_cap=bond_cap, fene_R0=20.0, nlist_cap=256, cell_cap=128,
                                   block_nlist=block)],
                    [dict(pos=pos, vel=np.zeros_like(pos), L=L, periodic=(0, 0, 0), n_cap=256,
                          bonds=np.array(pairs, dtype=np.int32))])
    # ghosts: the copies of tag 1 beside particle 0, and others
    g = np.concatenate([pos[0] + rng.uniform(-0.4, 0.4, (copies, 3)), 4.5 + 3.0 * rng.uniform(size=(40, 3))])
    gtag = np.concatenate([np.full(copies, 1), 1000 + np.arange(40)]).astype(np.int32)
    rec = np.zeros(len(g), dtype=[("pos", "<f8", 3), ("tag", "<i4"), ("pad", "<i4")])
    rec["pos"], rec["tag"] = g, gtag
    buf = torch.as_tensor(np.frombuffer(rec.tobytes(), dtype=np.uint8).copy(), device=ctx.device)
    ctx.unpack_ghosts(0, buf, len(g), B.FIELD_POS | B.FIELD_TAG, B.GHOST_SELECT, np.full(3, 100.0))
    ctx.build_nlist(True)
    ctx.check()
    assert ctx.general_tiles() == 0
    x = np.concatenate([pos, g])
    tag = np.concatenate([np.arange(n), gtag])
    partners = {}
    for a, b in pairs:
        partners.setdefault(a, set()).add(b)
        partners.setdefault(b, set()).add(a)
    nn, rows = ctx.neighbor_rows()
    for i in range(n):
        d2 = np.sum((x - x[i]) ** 2, axis=1)
        want = [j for j in np.nonzero(d2 < rl * rl)[0] if j != i and int(tag[j]) not in partners.get(i, ())]
        assert sorted(rows[i]) == want, i
