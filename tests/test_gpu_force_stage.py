"""GPU parity of the force pass where a tile's place in the launch or the
images of its halo are decided: more listed tiles than workgroups ahead, and
boxes in which a tile's half width + r_list is about half the box."""
import numpy as np
import pytest

from paper_1412_3387_amd import inputs
from tests.gpu_helpers import LJ, frel

pytestmark = pytest.mark.gpu

TOL = {0: 1e-12, 1: 1e-5}  # FP64; FP32 pair terms (6e-8 each, of forces tens of times the rms)


@pytest.fixture(scope="module")
def B():
    from paper_1412_3387_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("prec", [0, 1])
def test_more_rare_tiles_than_workgroups_ahead(orc, B, prec):
    """Shuffled rows of a 36,000-particle DPD fluid: all 563 tiles need
    per-pair images, more than the 512 workgroups that go ahead in the launch
    take, so every tile is done at its place."""
    big = inputs.dpd_fluid(36000, 61, 62)
    perm = np.random.default_rng(13).permutation(big.n)
    s = inputs.System(pos=big.pos[perm], vel=big.vel[perm], L=big.L, tag=perm.astype(np.int32))
    p = B.ModelParams(precision=prec, pair=B.PAIR_DPD, r_cut=1.0, r_buff=0.4, dt=0.02, dpd_A=25.0, dpd_gamma=4.5,
                      dpd_kT=1.0, dpd_seed=33, sort_period=0)
    out = []
    for mode in (B.FORCE_SPLIT, B.FORCE_ONE):
        p.force_launch = mode
        ctx = B.Context([p], [dict(pos=s.pos, vel=s.vel, L=s.L, tag=s.tag)])
        ctx.compute_forces(11, 0)
        ctx.check()
        assert ctx.rare_tiles() == 563
        out.append(ctx.host_state())
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    f, tag = out[0][2], out[0][3]
    fo = np.empty_like(f)
    fo[tag] = f
    which = np.sort(np.random.default_rng(14).choice(big.n, 256, replace=False))
    F, u, w, nc = orc.pair_forces("dpd", big.pos, big.L, [25.0, 4.5, 1.0, 1.0, 0.02, 33], vel=big.vel, tag=big.tag,
                                  timestep=11, which=which)
    fr = np.sqrt(np.mean(np.sum(F * F, axis=1)))
    assert np.max(np.sqrt(np.sum((fo[which, :3] - F) ** 2, axis=1))) / fr <= TOL[prec]


# boxes of three cells and a little more, where half the box minus r_list is
# about the half width of a tile: images around its centre or per pair
@pytest.mark.parametrize("n", [700, 1200, 2000, 2600, 3300, 4100, 6000])
@pytest.mark.parametrize("prec", [0, 1])
def test_small_box_images_after_drift(orc, B, n, prec):
    s = inputs.lj_fluid(n, n, n + 1)
    ctx = B.Context([B.ModelParams(precision=prec, sort_period=100)], [dict(pos=s.pos, vel=s.vel, L=s.L)])
    ctx.step(0, 33)  # up to r_buff / 2 away from the last build
    ctx.compute_forces(33, 0)
    ctx.check()
    x, v, f, tag = ctx.host_state()
    F, u, w, nc = orc.pair_forces("lj", x, s.L, LJ)
    assert frel(f[:, :3], F) <= TOL[prec]
