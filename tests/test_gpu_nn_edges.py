"""The network's convolution kernels at the edges of their tiles.

Reference: oracle/conv.py in FP64 on the same bfloat16-rounded weights.  The
kernels sum exact or FP32-rounded products in FP32, at most a few thousand
terms each, so 1e-5 of the largest value holds with room."""
import numpy as np
import pytest

from oracle import conv as C
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1906_11027_amd import sc_lbm as B  # noqa: E402


def _dev(a):
    return torch.tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


def _err(got, ref):
    return float(np.max(np.abs(got.cpu().numpy() - ref)) / np.max(np.abs(ref)))


# one row, a tile and one row past it; widths at, short of and past 16-pixel
# tiles (loaded 16 bytes or 4 at a time); channel counts of both kernels; one
# partial row, an odd and an even number, and more rows than tiles
@pytest.mark.parametrize("h,w", [(1, 32), (2, 33), (16, 16), (17, 15), (31, 48), (5, 2), (6, 5), (33, 46), (70, 40)])
@pytest.mark.parametrize("cin,cout", [(5, 32), (17, 32), (32, 32), (32, 1)])
@pytest.mark.parametrize("nblk", [1, 5, 300])
def test_weight_gradient_edges(h, w, cin, cout, nblk):
    rng = np.random.default_rng(h * 100 + w + cin)
    bsz = 2
    x = rng.normal(size=(bsz, cin, h, w)).astype(np.float32)
    g = rng.normal(size=(bsz, cout, h, w)).astype(np.float32)
    _, gw_ref, gb_ref = C.conv_bwd(x.astype(np.float64), np.zeros((cout, cin, 3, 3)), g.astype(np.float64))
    xd, gd = _dev(x), _dev(g)
    scratch = torch.empty(B.lib().sc_nn_bwd_weight_scratch_floats(cin, cout, nblk), device="cuda")
    gw, gb = torch.empty((cout, cin, 3, 3), device="cuda"), torch.empty(cout, device="cuda")
    assert B.lib().sc_nn_conv3x3_bwd_weight(xd.data_ptr(), gd.data_ptr(), scratch.data_ptr(), nblk, gw.data_ptr(),
                                            gb.data_ptr(), bsz, cin, cout, h, w,
                                            torch.cuda.current_stream().cuda_stream) == 0
    ew, eb = _err(gw, gw_ref), float(np.max(np.abs(gb.cpu().numpy() - gb_ref))) / np.max(np.sum(np.abs(g), (0, 2, 3)))
    say("weight gradient %d->%d %dx%d, %d rows: %.2e, bias %.2e" % (cin, cout, h, w, nblk, ew, eb))
    assert ew < 1e-5 and eb < 1e-6


# a strip of 32 pixels, one short of it, one and a half, narrow images; one to
# five rows (segments of every height); few and all channels
@pytest.mark.parametrize("h,w", [(1, 32), (2, 33), (3, 31), (5, 47), (4, 64), (9, 2), (1, 1), (70, 40)])
@pytest.mark.parametrize("cin", [1, 5, 17, 32])
def test_convolution_edges(h, w, cin):
    """Forward with and without tanh, and the input gradient with and without
    the tanh derivative (whose 32 output channels take cin channels of g)."""
    rng = np.random.default_rng(h * 100 + w + cin)
    bsz = 3
    bits = lambda a: torch.tensor(a, device="cuda").to(torch.bfloat16)   # noqa: E731
    x, bias = rng.normal(size=(bsz, cin, h, w)).astype(np.float32), rng.normal(size=32).astype(np.float32)
    wt = bits(rng.normal(scale=0.2, size=(32, cin, 3, 3)).astype(np.float32))
    ref = C.conv_fwd(x.astype(np.float64), wt.double().cpu().numpy(), bias.astype(np.float64))
    st = torch.cuda.current_stream().cuda_stream
    xd, bd, wd = _dev(x), _dev(bias), wt.view(torch.int16)
    out = torch.empty((bsz, 32, h, w), device="cuda")
    args = (xd.data_ptr(), wd.data_ptr(), bd.data_ptr(), out.data_ptr(), bsz, cin, 32, h, w, st)
    assert B.lib().sc_nn_conv3x3_fwd(*args) == 0
    e0 = _err(out, ref)
    assert B.lib().sc_nn_conv3x3_fwd_tanh(*args) == 0
    e1 = _err(out, np.tanh(ref))
    say("forward %d->32 %dx%d: %.2e, tanh %.2e" % (cin, h, w, e0, e1))
    assert e0 < 1e-5 and e1 < 1e-5
    if cin not in (1, 32):
        return
    # input gradient of a 32 -> cin layer
    wt = bits(rng.normal(scale=0.2, size=(cin, 32, 3, 3)).astype(np.float32))
    g, y = x, np.tanh(rng.normal(size=(bsz, 32, h, w))).astype(np.float32)
    ref, _, _ = C.conv_bwd(np.zeros((bsz, 32, h, w)), wt.double().cpu().numpy(), g.astype(np.float64))
    gd, yd, wd = _dev(g), _dev(y), wt.view(torch.int16)
    tmp = torch.empty(32 * 32 * 9, dtype=torch.int16, device="cuda")
    assert B.lib().sc_nn_conv3x3_bwd_data(gd.data_ptr(), wd.data_ptr(), tmp.data_ptr(), out.data_ptr(), bsz, 32, cin,
                                          h, w, st) == 0
    e0 = _err(out, ref)
    assert B.lib().sc_nn_conv3x3_bwd_data_tanh(gd.data_ptr(), wd.data_ptr(), tmp.data_ptr(), yd.data_ptr(),
                                               out.data_ptr(), bsz, 32, cin, h, w, st) == 0
    e1 = _err(out, ref * (1.0 - y.astype(np.float64) ** 2))
    say("input gradient 32->%d %dx%d: %.2e, tanh %.2e" % (cin, h, w, e0, e1))
    assert e0 < 1e-5 and e1 < 1e-5
