"""Grids of a few columns and 10^7 to 10^8 rows on the automatic shape.

A launch holds fewer than 2^32 threads a dimension.  Tiles 64 nodes wide with up
to 1,024 threads for 8 rows run out of that at 2^25 rows; these grids step on
two-dimensional blocks of at most 128 threads a row."""
import numpy as np
import pytest

from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1906_11027_amd import sc_lbm as B  # noqa: E402


@pytest.mark.parametrize("lattice,order,prec,rows,name", [
    ("D2Q9", 8, "fp32", 1 << 26, "tile64x16r4"), ("D2Q9", 10, "fp64", 1 << 27, "tile64x16r4"),
    ("D2Q13", 6, "fp32", 1 << 26, "wide128x16r2"), ("D2Q25", 8, "fp32", 1 << 26, "wide128x16r2"),
    ("D2Q25", 8, "fp64", 1 << 25, "wide64x8r2")])
def test_one_column(lattice, order, prec, rows, name):
    kw = dict(order=order, precision=prec, tau=0.9, forcing="guo" if lattice == "D2Q9" else "edm")
    h = B.sc_lbm_create(B.make_params(lattice, (1, rows), **kw))
    try:
        assert B.sc_lbm_variant_name(h) == name
        rc, done = B.sc_lbm_step(h, 3)
        say("%s E%d %s, 1 x %d: %s, %d steps" % (lattice, order, prec, rows, name, done))
        assert (rc, done) == (B.SC_OK, 3)
        o = B.sc_lbm_check(h)
        o = o[1] if isinstance(o, tuple) else o
        assert o.nonfinite == 0 and abs(o.mass / rows - 1.0) < 1e-6 and o.max_u < 1e-6
    finally:
        B.sc_lbm_destroy(h)
    torch.cuda.empty_cache()


def test_wide_grids_keep_their_shapes():
    """2^25 rows of 33 columns and more launch as before."""
    for shape in ((8192, 8192), (64, 65536)):
        h = B.sc_lbm_create(B.make_params("D2Q9", shape, order=8))
        assert B.sc_lbm_variant_name(h) == "tile2x64x16"
        B.sc_lbm_destroy(h)
