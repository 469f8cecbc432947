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
