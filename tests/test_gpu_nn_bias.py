"""Order of the bias gradient's sum in the layers with fewer than 32 channels.

The sum of a few hundred thousand values in FP32 is only as good as its order:
per 16 x 16 tile eight slices of 32 pixels (two tile rows), each slice's sum added
to the slice's running sum over a partial row's tiles, the eight slices as a tree,
then the rows (r = g mod 4 in four chains).  numpy's float32 adds the same values
in that order, and the kernel has to give its bits."""
import numpy as np
import pytest

from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1906_11027_amd import sc_lbm as B  # noqa: E402

F = np.float32


def _expected(g, nblk):
    """g [batch][cout][h][w]; nblk < 8 partial rows (row v: tiles v, v + nblk, ...)."""
    bsz, cout, h, w = g.shape
    ty, tx = -(-h // 16), -(-w // 16)
    pad = np.zeros((bsz, cout, 16 * ty, 16 * tx), F)
    pad[:, :, :h, :w] = g
    tiles = [pad[b, :, 16 * y:16 * y + 16, 16 * x:16 * x + 16] for b in range(bsz) for y in range(ty) for x in range(tx)]
    rows = []
    for v in range(nblk):
        acc = np.zeros((cout, 8), F)
        for t in tiles[v::nblk]:
            px = t.reshape(cout, 8, 32)
            s = np.zeros((cout, 8), F)
            for p in range(32):
                s = s + px[:, :, p]
            acc = acc + s
        a = acc[:, 0::2] + acc[:, 1::2]
        a = a[:, 0::2] + a[:, 1::2]
        rows.append(a[:, 0] + a[:, 1])
    part = [np.zeros(cout, F) for _ in range(4)]
    for v, r in enumerate(rows):
        part[v % 4] = part[v % 4] + r
    return ((part[0] + part[1]) + part[2]) + part[3]


@pytest.mark.parametrize("cin,cout", [(5, 32), (17, 32), (32, 1), (12, 1)])
@pytest.mark.parametrize("h,w", [(64, 96), (33, 46), (70, 15), (5, 3)])
@pytest.mark.parametrize("nblk", [1, 5])
def test_bias_order(cin, cout, h, w, nblk):
    bsz = 3
    rng = np.random.default_rng(h * 100 + w + cin)
    x = torch.tensor(rng.normal(size=(bsz, cin, h, w)).astype(F), device="cuda")
    g = rng.normal(size=(bsz, cout, h, w)).astype(F)
    gd = torch.tensor(g, device="cuda")
    scratch = torch.empty(B.lib().sc_nn_bwd_weight_scratch_floats(cin, cout, nblk), device="cuda")
    gw, gb = torch.empty((cout, cin, 3, 3), device="cuda"), torch.empty(cout, device="cuda")
    assert B.lib().sc_nn_conv3x3_bwd_weight(x.data_ptr(), gd.data_ptr(), scratch.data_ptr(), nblk, gw.data_ptr(),
                                            gb.data_ptr(), bsz, cin, cout, h, w,
                                            torch.cuda.current_stream().cuda_stream) == 0
    got, want = gb.cpu().numpy(), _expected(g, nblk)
    say("bias %d->%d %dx%d, %d rows: largest difference %.2e" % (cin, cout, h, w, nblk, np.max(np.abs(got - want))))
    assert np.array_equal(got, want)
