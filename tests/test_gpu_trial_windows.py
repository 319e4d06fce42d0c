"""One LM trial's sums where the members' windows are disjoint, nested, clipped
by the image or narrower than a tile's step, and at the member counts where the
evaluation changes its layout, against the FP64 oracle.  Tolerances as derived
for the Gram sums: J and r are rounded to FP32, 1e-6 of an entry's
Cauchy-Schwarz scale; F and chi2 are FP64 sums, 1e-9."""
import numpy as np
import pytest

import oracle
import skygen

pytestmark = pytest.mark.gpu

asp = pytest.importorskip("paper_1606_07872_amd")
pytest.importorskip("torch")

# (H, W), members (amplitude, x, y, sigma); widths 0.1 px from a window's step
WINDOWS = {
    "one pixel image": ((1, 1), [(0.7, 0.1, -0.2, 1.1)]),
    "three columns": ((700, 3), [(0.5, 1.2, 300.4, 30.1), (0.8, 0.7, 420.2, 17.1)]),
    "three rows": ((3, 700), [(0.5, 300.4, 1.2, 30.1), (0.8, 420.2, 0.7, 17.1)]),
    "disjoint": ((600, 500), [(0.6, 100.2, 90.3, 9.1), (0.4, 390.1, 470.4, 14.1)]),
    "small in large": ((512, 512), [(0.6, 250.2, 260.3, 2.1), (0.4, 240.1, 250.4, 40.1)]),
    "large holds small": ((512, 512), [(0.4, 240.1, 250.4, 40.1), (0.6, 250.2, 260.3, 2.1)]),
    "corner": ((300, 333), [(0.6, 2.2, 3.3, 12.1), (0.4, 331.1, 297.4, 25.1)]),
    "edges touch": ((400, 400), [(0.6, 150.0, 200.0, 10.1), (0.4, 253.0, 200.0, 10.1)]),
    "large shared": ((1500, 1400), [(0.6, 500.2, 600.3, 90.1), (0.4, 900.1, 800.4, 99.1)]),
}


def check(shape, th):
    H, W = shape
    th = np.asarray(th, dtype=np.float64)
    rng = np.random.default_rng(H * 31 + W)
    dirty = rng.normal(0.0, 0.3, size=shape).astype(np.float32)
    ctx = asp.Context(dirty, skygen.gaussian_psf(31, 3.0).astype(np.float32), 0.1, 0.0, max_iter=10,
                      max_active=16)
    st = th.copy()
    st[:, 0] *= 0.9
    st[:, 1] += 0.2
    st[0] = 0.0
    got = ctx.eval_trial(th, st)
    ab, wb = ctx.psf_gauss()
    o = oracle.Oracle(ctx.residual(), gain=0.1, max_iter=10, max_active=16, alpha_b=ab, omega_b=wb)
    ref = o.fit_eval(th, st)
    ctx.close()
    d = np.sqrt(np.maximum(np.diag(ref["H"]), 0.0))
    assert got["npx"] == ref["npx"]
    assert (np.abs(got["H"] - ref["H"]) <= 1e-6 * np.outer(d, d) + 1e-300).all()
    assert (np.abs(got["g"] - ref["g"]) <= 1e-6 * d * np.sqrt(ref["chi2"]) + 1e-300).all()
    assert abs(got["F"] - ref["F"]) <= 1e-9 * (abs(ref["F"]) + ref["chi2"])
    assert abs(got["chi2"] - ref["chi2"]) <= 1e-9 * ref["chi2"]


@pytest.mark.parametrize("name", list(WINDOWS))
def test_windows(name):
    check(*WINDOWS[name])


@pytest.mark.parametrize("m", [3, 4, 7, 8, 11, 12, 15, 16])
@pytest.mark.parametrize("sigma", [1.5, 12.0])
def test_member_counts(m, sigma):
    rng = np.random.default_rng(m)
    s = (np.floor(5 * rng.uniform(0.8, 1.2, size=m) * sigma) + 0.5) / 5.0
    xy = 200.0 + rng.uniform(-2, 2, size=(m, 2)) * sigma + 0.13
    check((400, 420), np.column_stack([rng.uniform(0.2, 1.0, size=m), xy, s]))
