"""The Gaussian of the PSF main lobe where the lobe meets the image's edges, is
one pixel, fills the image, or has a neighbour above the limit that is not
connected to it, against the oracle's fit of the same pixels."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

asp = pytest.importorskip("paper_1606_07872_amd")
pytest.importorskip("torch")


def gauss(H, W, cy, cx, s):
    y, x = np.mgrid[0:H, 0:W]
    return np.exp(-((y - cy) ** 2 + (x - cx) ** 2) / (2.0 * s * s)).astype(np.float32)


CASES = {
    "top left": gauss(40, 300, 0, 0, 3.0),
    "bottom right": gauss(37, 259, 36, 258, 4.0),
    "row wrap": gauss(20, 33, 9, 32, 2.5),
    "one pixel": np.maximum(gauss(64, 64, 30, 31, 0.2), 0.01).astype(np.float32),
    "fills": gauss(24, 18, 11, 9, 40.0),
    "two lobes": np.maximum(gauss(70, 300, 40, 100, 3.0), 0.9 * gauss(70, 300, 15, 140, 3.0)),
    "two peaks": np.maximum(gauss(64, 64, 20, 20, 2.0), gauss(64, 64, 40, 44, 2.0)),
    "more rows than threads": gauss(600, 17, 299, 8, 100.0),
}


@pytest.mark.parametrize("name", list(CASES))
def test_lobe(name):
    psf = CASES[name]
    dirty = np.zeros((64, 64), np.float32)
    dirty[30, 30] = 1.0
    ctx = asp.Context(dirty, psf, 0.1, 0.0, max_iter=1)
    ab, wb = ctx.psf_gauss()
    ao, wo = oracle.psf_fit(psf)[:2]
    assert abs(ab - ao) <= 1e-6 * abs(ao), (ab, ao)
    assert abs(wb - wo) <= 1e-6 * abs(wo), (wb, wo)
    ctx.close()
