"""run(n) on an image on either side of the size up to which the iterations of a
run share launches: the same components, count and stop as single steps."""
import numpy as np
import pytest

import skygen

pytestmark = pytest.mark.gpu

asp = pytest.importorskip("paper_1606_07872_amd")
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("H,W", [(8192, 65536), (8193, 65536)])
@pytest.mark.parametrize("tiles", [0, 1])
def test_run_is_steps(H, W, tiles):
    print("image", H, W, "tiles", tiles, flush=True)
    d = torch.zeros((H, W), device="cuda")
    k = torch.from_numpy(skygen.isolated_gaussian(25, 25, 1.0, 12.0, 12.0, 2.0).astype(np.float32))
    for i, (r, c) in enumerate([(0, 0), (H - 25, W - 25), (H // 2, W // 2), (100, W - 25)]):
        d[r:r + 25, c:c + 25] = (1.0 + i) * k.cuda()
    psf = torch.from_numpy(skygen.gaussian_psf(25, 3.0).astype(np.float32)).cuda()
    kw = dict(max_iter=50, max_active=1, peak_tiles=tiles)
    a = asp.Context(d, psf, 0.5, 0.9, **kw)
    b = asp.Context(d, psf, 0.5, 0.9, **kw)
    ra, rep = a.run(40)
    rb, n = 0, 0
    while rb == 0:
        rb = b.step()
        n += rb == 0
    assert ra == rb == asp.ASP_STOP_THRESHOLD and rep["iterations"] == n >= 8
    assert a.counts() == b.counts()
    assert np.array_equal(a.components_raw(), b.components_raw())
    assert a.residual_sumsq(True) == b.residual_sumsq(True)
    a.close()
    b.close()
