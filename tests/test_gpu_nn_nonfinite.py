"""Infinite inputs of the layers with fewer than 32 channels: a product with an
infinite value is infinite, and partial rows that have no tile add nothing to it."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover
    pytest.skip("no GPU", allow_module_level=True)

from paper_1906_11027_amd import sc_lbm as B  # noqa: E402


@pytest.mark.parametrize("cin,cout", [(5, 32), (12, 1), (32, 1), (17, 32)])
@pytest.mark.parametrize("bsz", [1, 2, 3])
@pytest.mark.parametrize("nblk", [1, 2, 4, 5])
def test_infinite_input(cin, cout, bsz, nblk):
    """One infinite pixel in the last image's only tile: every weight of its
    channel is infinite, with the sign of the gradient that it meets."""
    rng = np.random.default_rng(cin + nblk)
    x = rng.normal(size=(bsz, cin, 16, 16)).astype(np.float32)
    g = rng.normal(size=(bsz, cout, 16, 16)).astype(np.float32)
    ci, y, c = cin - 2, 6, 9
    x[-1, ci, y, c] = np.inf
    xd, gd = torch.tensor(x, device="cuda"), torch.tensor(g, device="cuda")
    scratch = torch.empty(B.lib().sc_nn_bwd_weight_scratch_floats(cin, cout, nblk), device="cuda")
    gw, gb = torch.empty((cout, cin, 3, 3), device="cuda"), torch.empty(cout, device="cuda")
    assert B.lib().sc_nn_conv3x3_bwd_weight(xd.data_ptr(), gd.data_ptr(), scratch.data_ptr(), nblk, gw.data_ptr(),
                                            gb.data_ptr(), bsz, cin, cout, 16, 16,
                                            torch.cuda.current_stream().cuda_stream) == 0
    got = gw.cpu().numpy()
    for dy in range(3):
        for dx in range(3):
            want = np.sign(g[-1, :, (y + 1 - dy) % 16, (c + 1 - dx) % 16]) * np.inf
            assert np.array_equal(got[:, ci, dy, dx], want), (dy, dx)
    assert np.isfinite(np.delete(got, ci, 1)).all()
