"""A run whose iterations are long: its launches end after 10 ms, long before
their 32 iterations, with the result of single steps bit for bit, and a call on
another stream that needs a CU's LDS gets its turn between them."""
import threading
import time

import numpy as np
import pytest

import skygen
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

asp = pytest.importorskip("paper_1606_07872_amd")
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def wide():
    """Components of hundreds of pixels: some 2 ms an iteration."""
    n = 4096
    g = torch.Generator(device="cuda").manual_seed(3)
    y, x = torch.meshgrid(torch.arange(n, device="cuda").float(),
                          torch.arange(n, device="cuda").float(), indexing="ij")
    d = torch.exp(-((y - 2000) ** 2 + (x - 2100) ** 2) / (2 * 500.0 ** 2))
    d += 0.7 * torch.exp(-((y - 1000) ** 2 + (x - 3100) ** 2) / (2 * 400.0 ** 2))
    return d + 1e-3 * torch.randn((n, n), device="cuda", generator=g)


def context(d):
    psf = torch.from_numpy(skygen.gaussian_psf(25, 3.0).astype(np.float32)).cuda()
    return asp.Context(d, psf, 0.1, 0.0, max_iter=2000, max_active=2, max_width=1000.0)


def test_long_run_is_steps(wide):
    a, b = context(wide), context(wide)
    rc, rep = a.run(40)
    assert rc == asp.ASP_OK and rep["iterations"] == 40
    for _ in range(40):
        assert b.step() == asp.ASP_OK
    assert a.counts() == b.counts()
    assert np.array_equal(a.residual(), b.residual())
    assert np.array_equal(a.components_raw(), b.components_raw())
    a.close()
    b.close()


def test_another_stream_gets_its_turn(wide):
    c = context(wide)
    net = asp.Mlp(omlp.init_params(np.random.default_rng(0)).astype(np.float32), max_batch=1)
    x = torch.zeros((64, 1024), device="cuda")
    y = torch.zeros((64, 4), device="cuda")
    net.forward(x, y)
    c.run(8)
    t = time.perf_counter()
    c.run(64)
    whole = (time.perf_counter() - t) / 2          # 32 iterations
    assert whole > 0.03
    run = threading.Thread(target=c.run, args=(128,))
    waits = []
    run.start()
    while run.is_alive():
        t = time.perf_counter()
        net.forward(x, y)
        waits.append(time.perf_counter() - t)
    run.join()
    print(f"32 iterations {1e3 * whole:.1f} ms, {len(waits)} calls, median wait "
          f"{1e3 * np.median(waits):.1f} ms", flush=True)
    assert np.median(waits) < whole / 2
    net.close()
    c.close()
