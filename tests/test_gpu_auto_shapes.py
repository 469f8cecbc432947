"""Lines of the automatic 2D launch shapes where both sides were measured (the
figures stand at the rules in sc_lbm.cpp): the shape on either side of each."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1906_11027_amd import sc_lbm as B  # noqa: E402


@pytest.mark.parametrize("lattice,forcing,prec,order,shape,name", [
    # E10 in FP64: a mostly empty last round of 32 x 32 tiles goes to one step
    ("D2Q9", "guo", "fp64", 10, (504, 504), "tile2x32x32"), ("D2Q9", "guo", "fp64", 10, (529, 529), "tile32x8r1"),
    ("D2Q9", "guo", "fp64", 10, (567, 493), "tile32x8r1"), ("D2Q9", "guo", "fp64", 10, (640, 640), "tile2x32x32"),
    ("D2Q9", "guo", "fp64", 10, (721, 721), "tile32x8r1"), ("D2Q9", "guo", "fp64", 10, (2048, 2048), "tile2x32x32"),
    # E10 in FP32: 64 x 16, 32 x 32 only where it fills two rounds
    ("D2Q9", "guo", "fp32", 10, (500, 500), "tile2x64x16"), ("D2Q9", "guo", "fp32", 10, (1224, 408), "tile2x32x32"),
    ("D2Q9", "guo", "fp32", 10, (774, 774), "tile2x64x16"), ("D2Q9", "guo", "fp32", 10, (1702, 1702), "tile2x64x16"),
    ("D2Q9", "guo", "fp32", 10, (3331, 1110), "tile2x64x16"), ("D2Q9", "guo", "fp32", 10, (2048, 2048), "tile2x64x16"),
    # D2Q9 with the exact difference method: 64 x 16 at every order
    ("D2Q9", "edm", "fp32", 10, (1732, 1732), "wide2x64x16t1024"), ("D2Q9", "edm", "fp32", 8, (1732, 1732), "wide2x64x16t1024"),
    # D2Q13 E10 in FP32: one step while both copies of the state fit the cache
    ("D2Q13", "edm", "fp32", 10, (1516, 1516), "wideK1x16x16"), ("D2Q13", "edm", "fp32", 10, (1702, 1702), "wide2x64x8t1024"),
    ("D2Q13", "edm", "fp32", 10, (2000, 2000), "wide2x64x8t1024"),
    ("D2Q13", "edm", "fp32", 10, (748, 1902), "wide128x16r2"), ("D2Q13", "guo", "fp32", 10, (958, 2298), "wide128x16r2"),
    ("D2Q13", "edm", "fp32", 10, (1500, 1500), "wideK1x16x16"), ("D2Q13", "edm", "fp32", 10, (160, 9000), "wideK1x16x16"),
    # D2Q25 from E6 and D2Q13 E6, E8 in FP64: one step in the cache
    ("D2Q25", "edm", "fp32", 8, (1148, 1148), "wideK1x64x8"), ("D2Q25", "edm", "fp32", 8, (1166, 1166), "wide128x16r2"),
    ("D2Q25", "edm", "fp32", 8, (1216, 1216), "wide2x64x16t1024"), ("D2Q25", "edm", "fp64", 8, (728, 728), "wideK1x16x16"),
    ("D2Q25", "edm", "fp64", 6, (68, 8235), "wide32x8r1"), ("D2Q25", "edm", "fp64", 8, (830, 830), "wideK1x64x8"),
    ("D2Q13", "edm", "fp64", 8, (1131, 1131), "wideK1x16x16"), ("D2Q13", "edm", "fp64", 8, (1144, 1144), "wide2x64x12t768"),
    # strips that the tiles hang over, and their neighbours that they do not
    ("D2Q13", "edm", "fp32", 8, (70, 12857), "wideK1x16x16"), ("D2Q13", "edm", "fp32", 8, (24, 16666), "wide32x8r1"),
    ("D2Q13", "edm", "fp32", 8, (192, 4700), "wide2x64x12t768"), ("D2Q25", "edm", "fp32", 4, (88, 10227), "wideK1x16x16"),
    ("D2Q25", "edm", "fp32", 4, (128, 7000), "wide2x64x8t512"), ("D2Q9", "edm", "fp64", 6, (131, 6870), "wideK1x16x16"),
    ("D2Q9", "edm", "fp64", 6, (34, 11764), "wideK1x16x16"), ("D2Q9", "edm", "fp64", 6, (128, 6870), "wide2x64x8t512"),
    ("D2Q13", "edm", "fp64", 8, (88, 1704), "wideK1x16x16"), ("D2Q13", "edm", "fp64", 8, (24, 3333), "wide32x8r1"),
    ("D2Q25", "edm", "fp64", 4, (70, 5714), "wide32x8r1"), ("D2Q25", "edm", "fp64", 4, (96, 5714), "wide2x32x8t256"),
    ("D2Q25", "edm", "fp64", 8, (49, 4489), "wide32x8r1"),
    # D2Q9 strips off the multiples of 64, from 1.5 million nodes
    ("D2Q9", "guo", "fp32", 8, (451, 5276), "tile64x16r4"), ("D2Q9", "guo", "fp32", 8, (448, 5276), "tile2x64x16"),
    ("D2Q9", "guo", "fp32", 10, (313, 10523), "tile64x16r4"), ("D2Q9", "guo", "fp32", 6, (513, 4745), "tile2x64x16"),
    ("D2Q9", "guo", "fp32", 8, (451, 2400), "tile2x64x16"), ("D2Q9", "guo", "fp32", 8, (451, 9000), "tile2x64x16"),
    ("D2Q9", "edm", "fp32", 6, (210, 17276), "wide128x16r2"), ("D2Q9", "edm", "fp32", 8, (388, 5154), "wide2x64x16t1024"),
])
def test_shape(lattice, forcing, prec, order, shape, name):
    h = B.sc_lbm_create(B.make_params(lattice, shape, order=order, precision=prec, forcing=forcing, tau=0.9))
    try:
        assert B.sc_lbm_variant_name(h) == name
    finally:
        B.sc_lbm_destroy(h)
