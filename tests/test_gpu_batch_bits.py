"""The batched sweep's results to the bit, over its launch shapes and precisions.

A droplet that blows up is retired at the next check, finite on some of its
nodes and not on others; which ones hangs on the rounding of every step before.
So a change of the order of operations, harmless to every stable droplet, gives
such an item another field.  golden/batch_bits.json holds what the batch kernels
gave on gfx950 with ROCm 7.2 before the single grids' steps got an order of
operations of their own.  The shape of 32 x 8 tiles (1) follows the single
grids."""
import json
import os

import numpy as np
import pytest

from tests import batch_bits
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1906_11027_amd import Sim  # noqa: E402
from paper_1906_11027_amd.sc_lbm import Batch  # noqa: E402

with open(os.path.join(os.path.dirname(__file__), "golden", "batch_bits.json")) as f:
    GOLD = json.load(f)


@pytest.mark.parametrize("shape", [-1, 0, 2, 3])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_sweep_bits(prec, shape):
    got = batch_bits.sweep(Batch, prec, shape)
    for it, g, want in zip(batch_bits.ITEMS, got, GOLD["%s %d" % (prec, shape)]):
        say("%s shape %d, %s: steps, rule, non-finite, CRC %s" % (prec, shape, it, g))
        assert g == want, (it, g, want)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_small_tiles_follow_the_single_grid(prec):
    """An item on 32 x 8 tiles and a run of its own on tile2x32x8 (variant 10)."""
    items = [dict(rho0=batch_bits.density(s), order=o, G=g, tau=t, init=i) for s, o, g, t, i in batch_bits.ITEMS]
    bt = Batch(items, precision=prec, variant=1)
    bt.step(90)
    for k, it in enumerate(items):
        one = Sim(it.pop("rho0"), "D2Q9", precision=prec, variant=10, rho_ref=bt.rho_ref, **it)
        one.step(90)
        assert one.variant == "tile2x32x8"
        assert np.array_equal(one.observe()["rho"], bt.observe(k)["rho"], equal_nan=True), batch_bits.ITEMS[k]
        one.close()
    bt.close()
