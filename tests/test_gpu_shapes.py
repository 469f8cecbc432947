"""Launch shapes chosen by a rule, against the plain shapes of the same step.

The shapes do the same arithmetic on the same values; on D3Q19 the compiler may
fuse multiply-adds differently per shape, so there the states agree after k
steps to a few roundings of their largest value per step (2e-6 in FP32 and 1e-14 in FP64
relative to it over 6 steps)."""
import numpy as np
import pytest

from tests.gpu_helpers import say
from workload import droplet_rho

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1906_11027_amd import Sim  # noqa: E402
from paper_1906_11027_amd import sc_lbm as B  # noqa: E402


def _state(rho0, lattice, steps, prec, variant, **kw):
    sim = Sim(rho0, lattice, precision=prec, variant=variant, **kw)
    sim.step(steps)
    st, name = sim.state().astype(np.float64), sim.variant
    sim.close()
    return st, name


def _agree(rho0, lattice, steps, prec, variant, plain, **kw):
    st, name = _state(rho0, lattice, steps, prec, variant, **kw)
    ref, rname = _state(rho0, lattice, steps, prec, plain, **kw)
    d, top = float(np.max(np.abs(st - ref))), float(np.max(np.abs(ref)))
    say("%s %s %s: %s vs %s max |diff| %.2e of %.2e" % (lattice, rho0.shape, prec, name, rname, d, top))
    assert d <= (2e-6 if prec == "fp32" else 1e-14) * top


# grids thinner than the psi window, one column, many columns, and a height
# that the segments do not divide
@pytest.mark.parametrize("shape", [(9, 7, 1), (33, 9, 2), (20, 17, 5), (70, 9, 131), (300, 40, 11)])
@pytest.mark.parametrize("order,collision", [(4, "srt"), (8, "mrt")])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_balanced_march(shape, order, collision, prec):
    """D3Q19 persistent marches with the balanced segment height (the
    automatic shape and both tiles) against march32x8h16."""
    rho0 = droplet_rho(shape, 3, seed=4)
    n = B.sc_lbm_num_variants(B.make_params("D3Q19", shape))
    for v in (-1, n - 2, n - 1):
        _agree(rho0, "D3Q19", 6, prec, v, 2, order=order, collision=collision, tau=0.9)


# sizes on either side of each line of the 2D rule; 5 steps: two two-step
# launches and the single step of the remainder
@pytest.mark.parametrize("shape", [(60, 40), (331, 332), (410, 390), (1030, 520), (1300, 1160)])
@pytest.mark.parametrize("lattice", ["D2Q9", "D2Q9edm", "D2Q13", "D2Q25"])
@pytest.mark.parametrize("order", [4, 8, 10])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_automatic_2d_shape(shape, lattice, order, prec):
    """The automatic 2D shape against a one-step shape of the same family
    (tile64x8r2 / wide32x8r1)."""
    rho0 = droplet_rho(shape, 13, seed=5)
    edm = lattice != "D2Q9"
    _agree(rho0, lattice.replace("edm", ""), 5, prec, -1, 1, order=order, tau=0.9, forcing="edm" if edm else "guo")


@pytest.mark.parametrize("lattice", ["D2Q9", "D2Q9edm", "D2Q13", "D2Q25"])
@pytest.mark.parametrize("order", [4, 6, 8, 10])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_2d_steps_round_alike(lattice, order, prec):
    """Every 2D launch shape, and a run cut into single steps, gives the same
    bits: 7 steps are three two-step launches and one single step."""
    rho0 = droplet_rho((60, 44), 13, seed=6)
    kw = dict(order=order, tau=0.9, forcing="edm" if lattice != "D2Q9" else "guo", precision=prec)
    lat = lattice.replace("edm", "")
    one = Sim(rho0, lat, **kw)
    for _ in range(7):
        one.step(1)
    want = one.state()
    one.close()
    for v in range(-1, B.sc_lbm_num_variants(B.make_params(lat, (60, 44), **kw))):
        sim = Sim(rho0, lat, variant=v, **kw)
        sim.step(7)
        assert np.array_equal(sim.state(), want), (v, sim.variant)
        sim.close()


# one node per thread: grids narrower than the halo of four steps, one tile and
# a node more, a ragged grid of many tiles
@pytest.mark.parametrize("shape", [(3, 2), (1, 17), (9, 33), (75, 130)])
@pytest.mark.parametrize("lattice", ["D2Q9", "D2Q9edm", "D2Q13", "D2Q25"])
@pytest.mark.parametrize("walls", [False, True])
@pytest.mark.parametrize("order,prec", [(4, "fp32"), (8, "fp64"), (10, "fp32")])
def test_steps_per_launch_round_alike(shape, lattice, walls, order, prec):
    """Shapes of one, two and four steps per launch, with and without walls:
    7 steps at once give the bits of 7 single steps of the plain tile."""
    rng = np.random.default_rng(7)
    rho0 = 1.0 + 0.05 * rng.random(shape)
    solid = (rng.random(shape) < 0.2).astype(np.uint8) if walls else None
    kw = dict(order=order, tau=0.9, forcing="edm" if lattice != "D2Q9" else "guo", precision=prec)
    lat = lattice.replace("edm", "")
    states = []
    count = B.sc_lbm_num_variants(B.make_params(lat, shape, **kw))
    for v in [1, -1] + list(range(count)):
        sim = Sim(rho0, lat, variant=v, **kw)
        if walls:
            sim.set_walls(solid, 0.8)
        for k in [1] * 7 if not states else [7]:
            sim.step(k)
        states.append((sim.state(), v, sim.variant))
        sim.close()
    for state, v, name in states[1:]:
        assert np.array_equal(state, states[0][0]), (v, name)
