"""GPU parity of the Morton sort around the sizes where its path changes: one
radix tile of 1,024 rows, and 64 of them, above which the digit counts are
scanned by launches of their own."""
import numpy as np
import pytest

from paper_1412_3387_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1412_3387_amd import binding
    binding.lib()
    return binding


def _spread(v):
    out = np.zeros_like(v)
    for b in range(10):
        out |= ((v >> b) & 1) << (3 * b)
    return out


def _order(pos, L):
    """Stable order of the 30-bit Morton codes, 10 bits per axis."""
    q = np.clip(np.floor(pos * (1024.0 / L)), 0, 1023).astype(np.int64)
    return np.argsort(_spread(q[:, 0]) | _spread(q[:, 1]) << 1 | _spread(q[:, 2]) << 2, kind="stable")


@pytest.mark.parametrize("sizes", [(1,), (63,), (1023, 64), (1024,), (1025,), (40000,), (65472,), (65536,), (65537,),
                                   (70000,), (30000, 1, 36000), (500, 70000, 3)])
@pytest.mark.parametrize("bonded", [False, True])
def test_rows_in_morton_order(B, sizes, bonded):
    rng = np.random.default_rng(sum(sizes))
    systems = []
    for n in sizes:
        L = np.array([max(9.0, (n / 0.4) ** (1 / 3)), max(8.0, (n / 0.4) ** (1 / 3)), max(7.0, (n / 0.4) ** (1 / 3))])
        sy = dict(pos=rng.uniform(0, 1, (n, 3)) * L, vel=rng.normal(size=(n, 3)), L=L)
        sy["bonds"] = np.stack([np.arange(0, n - 1, 2), np.arange(1, n, 2)], axis=1).astype(np.int32) if bonded else None
        systems.append(sy)
    p = B.ModelParams(precision=B.FP64, sort_period=1, nlist_cap=160, bond_cap=2 if bonded else 0, fene_R0=400.0)
    ctx = B.Context([p] * len(sizes), systems)
    ctx.build_nlist(True)
    ctx.check()
    for k, sy in enumerate(systems):
        want = _order(sy["pos"], sy["L"])
        x, v, f, tag = ctx.host_state(k)
        assert np.array_equal(tag, want)
        assert np.array_equal(x, sy["pos"][want]) and np.array_equal(v, sy["vel"][want])
    if bonded:
        # the partners moved with their rows: nothing excluded is listed
        nn, rows = ctx.neighbor_rows(0)
        tag = ctx.host_state(0)[3]
        for r in range(min(len(tag), 2000)):
            t = tag[r]
            other = t + 1 if t % 2 == 0 else t - 1
            assert other not in tag[rows[r]]
