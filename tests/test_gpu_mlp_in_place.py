"""A forward pass whose outputs take the place of the first inputs, or of inputs
that an earlier part of the pass has read: the same outputs as with arrays of
their own, on both routes and at the seams of the parts."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

asp = pytest.importorskip("paper_1606_07872_amd")
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n,bmax", [(64, 64), (65, 64), (700, 1), (4097, 512), (5000, 4096)])
@pytest.mark.parametrize("at", [0, 4])
def test_outputs_over_inputs(n, bmax, at):
    rng = np.random.default_rng(n)
    net = asp.Mlp(omlp.init_params(rng).astype(np.float32), max_batch=bmax)
    X = rng.normal(0.0, 0.3, size=(n, 1024)).astype(np.float32)
    x = torch.from_numpy(X).cuda()
    want = torch.empty((n, 4), dtype=torch.float32, device="cuda")
    net.forward(x, want)
    # outputs from float `at` of the inputs on: row r's lie within inputs 0 .. r
    y = x.view(-1)[at:at + 4 * n].view(n, 4)
    net.forward(x, y)
    assert torch.equal(y, want)
    net.close()
