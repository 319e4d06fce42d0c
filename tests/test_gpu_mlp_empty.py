"""A forward pass of no rows: accepted, with and without arrays, and nothing is
written; the network serves the next call as before."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

asp = pytest.importorskip("paper_1606_07872_amd")
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bmax", [1, 64])
def test_forward_of_no_rows(bmax):
    rng = np.random.default_rng(5)
    net = asp.Mlp(omlp.init_params(rng).astype(np.float32), max_batch=bmax)
    x = torch.from_numpy(rng.normal(0.0, 0.3, size=(1, 1024)).astype(np.float32)).cuda()
    y = torch.full((1, 4), 7.0, dtype=torch.float32, device="cuda")
    L = asp.lib()
    assert L.asp_mlp_forward(net._n, None, 0, None) == asp.ASP_OK
    assert L.asp_mlp_forward(net._n, x.data_ptr(), 0, y.data_ptr()) == asp.ASP_OK
    assert (y.cpu().numpy() == 7.0).all()
    net.forward(x, y)
    want, _ = omlp.forward(net.weights(), x.cpu().numpy())
    assert np.abs(y.cpu().numpy() - want).max() <= 1e-4
    net.close()
