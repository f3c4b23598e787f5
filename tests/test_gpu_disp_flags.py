"""GPU parity of the one-launch displacement check of a single system: whether
the list is rebuilt when one particle, wherever its row, has moved."""
import pytest

from paper_1412_3387_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1412_3387_amd import binding
    binding.lib()
    return binding


# one workgroup and part of one, 256 of them and more rows than they take at once
@pytest.mark.parametrize("n", [600, 1024, 1025, 65536, 65537, 70000])
def test_one_moved_particle_rebuilds(B, n):
    s = inputs.lj_fluid(n, 3, 4, density=0.5)
    ctx = B.Context([B.ModelParams(precision=B.FP64, r_buff=0.4)], [dict(pos=s.pos, vel=s.vel, L=s.L)])
    ctx.build_nlist(True)
    for row in (0, n // 2, n - 1):
        for step, rebuilt in ((0.19, 0), (0.02, 1), (0.0, 0)):
            before = ctx.build_count()
            ctx.pos[row, 0] = (ctx.pos[row, 0] + step) % float(s.L[0])
            ctx.build_nlist(False)
            ctx.check()
            assert ctx.build_count() - before == rebuilt, (row, step)
