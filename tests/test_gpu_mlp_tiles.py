"""The network's products at the edges of their tiles: batches that fill,
miss and overhang the 32-row and 16-row tiles, picked rows, inputs that start
off a 16-byte boundary, and both routes of the forward pass, against FP64."""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

asp = pytest.importorskip("paper_1606_07872_amd")
torch = pytest.importorskip("torch")

U = 2.0 ** -24


def rows(rng, n, cols, shift):
    """n x cols normal values and a device view of them that starts `shift` floats
    past an aligned allocation."""
    a = rng.normal(0.0, 0.3, size=(n, cols)).astype(np.float32)
    buf = torch.zeros(n * cols + shift, dtype=torch.float32, device="cuda")
    buf[shift:] = torch.from_numpy(a.ravel()).cuda()
    return a.astype(np.float64), buf[shift:].view(n, cols)


def forward_with_bound(w, X):
    """FP64 outputs and a bound on the error of FP32 sums in any order."""
    W1, b1, W2, b2, W3, b3 = omlp.unpack(w)
    h, e = X, np.zeros_like(X)
    for W, b, last in ((W1, b1, False), (W2, b2, False), (W3, b3, True)):
        k = W.shape[1]
        a = np.abs(h) + e
        e = e @ np.abs(W).T + (k + 2) * U * (a @ np.abs(W).T + np.abs(b))
        h = h @ W.T + b
        if not last:
            h = np.maximum(h, 0.0)
    return h, e


@pytest.mark.parametrize("n,bmax,shift", [
    (1, 64, 0), (16, 16, 1), (17, 64, 0), (33, 64, 3), (65, 64, 0), (66, 64, 1),
    (3072, 3072, 0), (3073, 3073, 2), (4097, 512, 0), (13 * 16 * 256 + 5, 64, 0)])
def test_forward_edges(n, bmax, shift):
    rng = np.random.default_rng(n)
    w = omlp.init_params(rng).astype(np.float32)
    X, xd = rows(rng, n, 1024, shift)
    net = asp.Mlp(w, max_batch=bmax)
    y = torch.full((n, 4), 7.0, dtype=torch.float32, device="cuda")
    net.forward(xd, y)
    want, bound = forward_with_bound(w.astype(np.float64), X)
    assert (np.abs(y.cpu().numpy() - want) <= bound).all()
    net.close()


@pytest.mark.parametrize("B,shift", [(1, 0), (15, 1), (32, 0), (65, 3), (511, 0), (530, 1)])
def test_step_edges(B, shift):
    """One batch of picked rows, in order and repeated: the gradient (read back
    from a batch of the same rows) to the 1e-4 of each tensor that FP32 gives,
    and the loss of a training step."""
    rng = np.random.default_rng(B)
    w = omlp.init_params(rng).astype(np.float32)
    n = 97
    X, xd = rows(rng, n, 1024, shift)
    T, td = rows(rng, n, 4, shift)
    pick = rng.integers(0, n, size=B)
    w64 = w.astype(np.float64)
    lo, go = omlp.loss_and_grad(w64, X[pick], T[pick])
    net = asp.Mlp(w, max_batch=B)
    idx = torch.from_numpy(pick).cuda()
    loss, g = net.loss_grad(xd[idx].contiguous(), td[idx].contiguous())
    assert abs(loss - lo) <= 1e-5 * lo
    for a, b in zip(omlp.unpack(g.astype(np.float64)), omlp.unpack(go)):
        assert np.abs(a - b).max() <= 1e-4 * np.abs(b).max()
    mean = net.train(xd, td, idx.to(torch.int32), B, 1e-3)
    assert abs(mean - lo) <= 1e-5 * lo
    # the picked rows and the same rows laid out give the same step, bit for bit
    other = asp.Mlp(w, max_batch=B)
    other.train(xd[idx].contiguous(), td[idx].contiguous(),
                torch.arange(B, dtype=torch.int32, device="cuda"), B, 1e-3)
    assert (net.weights() == other.weights()).all()
    net.close()
    other.close()
