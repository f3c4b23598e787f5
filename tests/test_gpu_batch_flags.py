"""A batch of more systems than the list of rebuilt systems takes in one go
(256), of which a few rebuild at a time: trajectories against single systems."""
import numpy as np
import pytest

from paper_1412_3387_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1412_3387_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("prec", [0, 1])
def test_many_small_systems_rebuild_apart(B, prec):
    """300 systems of 60 to 400 particles (tiles that need per-pair images
    among them), each with a speed of its own so that they rebuild at
    different steps; one without particles between them."""
    rng = np.random.default_rng(3)
    systems = []
    for k in range(300):
        s = inputs.lj_fluid(int(rng.integers(60, 400)), 100 + k, 500 + k, density=0.25)
        systems.append(dict(pos=s.pos, vel=s.vel * (0.3 + 0.01 * k), L=s.L))
    systems[270] = dict(pos=np.zeros((0, 3)), vel=np.zeros((0, 3)), L=np.full(3, 9.0))
    p = B.ModelParams(precision=prec, tpp_force=4, sort_period=25)
    ctx = B.Context([p] * 300, systems)
    ctx.step(0, 60)
    ctx.check()
    for k in (0, 3, 77, 255, 256, 257, 269, 271, 299):
        one = B.Context([p], [systems[k]])
        one.step(0, 60)
        one.check()
        for a, b in zip(ctx.host_state(k), one.host_state()):
            assert np.array_equal(a, b), k
