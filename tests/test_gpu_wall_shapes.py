"""The launch shape of handles with walls: what they report is what runs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1906_11027_amd import Sim  # noqa: E402
from paper_1906_11027_amd import sc_lbm as B  # noqa: E402


def _channel(shape):
    solid = np.zeros(shape, dtype=np.uint8)
    solid[:, :2] = solid[:, -2:] = 1
    return solid


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(60, 44), (400, 300)])
def test_name_and_steps_describe_one_shape(shape, prec):
    """Each two-step shape of several nodes a thread ("wide2x...") has no wall
    form: with walls the handle names the one that it runs, and without them its
    own again."""
    kw = dict(order=8, tau=0.9, forcing="edm", precision=prec)
    for v in range(B.sc_lbm_num_variants(B.make_params("D2Q13", shape, **kw))):
        sim = Sim(np.ones(shape), "D2Q13", variant=v, **kw)
        name, steps = sim.variant, sim.steps_per_launch
        sim.set_walls(_channel(shape), 1.0)
        with_walls, k = sim.variant, sim.steps_per_launch
        assert not with_walls.startswith("wide2x"), (name, with_walls)
        if not name.startswith("wide2x"):
            assert (with_walls, k) == (name, steps)
        # the name's number of steps, where it has one, is the most that it takes
        most = int(with_walls[5]) if with_walls.startswith("wideK") else 1
        assert 1 <= k <= most, (with_walls, k)
        sim.set_walls(None, 0.0)
        assert (sim.variant, sim.steps_per_launch) == (name, steps)
        sim.close()


@pytest.mark.parametrize("order", [4, 6, 8, 10])
def test_large_d2q25_fp64_does_not_spill(order):
    """From 2^20 nodes D2Q25 in FP64 steps on 512-thread or one-node tiles, with
    walls too: the 1,024-thread blocks of wide128x16r2 spill its 25 values.  An odd
    step more than the launches take gives the bits of single steps."""
    shape = (1030, 1024)
    rho0 = 1.0 + 0.05 * np.random.default_rng(3).random(shape)
    kw = dict(order=order, tau=0.9, forcing="edm", precision="fp64")
    sim = Sim(rho0, "D2Q25", **kw)
    sim.set_walls(_channel(shape), 1.0)
    assert sim.variant in ("wide64x8r2", "wideK1x64x8"), sim.variant
    sim.set_walls(None, 0.0)
    one = Sim(rho0, "D2Q25", variant=1, **kw)
    sim.step(3)
    one.step(3)
    assert np.array_equal(sim.state(), one.state())
    sim.close()
    one.close()


def test_flat_channel_takes_tiles_that_fit():
    """5586 x 38: 16 x 16 tiles cover a quarter more than the grid, 32 x 8 tiles 5%."""
    for shape, name in (((5586, 38), "wide32x8r1"), ((5600, 48), "wideK1x16x16")):
        sim = Sim(np.ones(shape), "D2Q9", order=8)
        sim.set_walls(_channel(shape), 1.0)
        assert sim.variant == name, (shape, sim.variant)
        sim.close()


def test_fp64_strips_that_16_rows_hang_over():
    """33 rows: 16 x 16 tiles cover 48 of them, 8-row tiles 40."""
    shape = (2760, 33)
    sim = Sim(np.ones(shape), "D2Q9", order=10, tau=0.9, precision="fp64")
    sim.set_walls(_channel(shape), 1.0)
    assert sim.variant == "wide32x8r1", sim.variant
    sim.close()
