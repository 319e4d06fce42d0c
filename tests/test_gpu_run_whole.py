"""run(n), whose iterations share launches, against n single steps, each step
with its own launches: the same residual, components, counts and stop, bit for
bit, at run lengths around the iterations of a launch, over several calls, with
both peak searches, and through each stop."""
import numpy as np
import pytest

import skygen

pytestmark = pytest.mark.gpu

asp = pytest.importorskip("paper_1606_07872_amd")
pytest.importorskip("torch")


def field(H, W):
    rng = np.random.default_rng(H * 1000 + W)
    y, x = np.mgrid[0:H, 0:W]
    d = rng.normal(0.0, 0.01, size=(H, W))
    for _ in range(max(1, H * W // 600)):
        cy, cx, s = rng.uniform(0, H), rng.uniform(0, W), rng.uniform(1.3, 4.0)
        d += rng.uniform(0.2, 1.0) * np.exp(-((y - cy) ** 2 + (x - cx) ** 2) / (2 * s * s))
    return d.astype(np.float32)


def context(d, **kw):
    return asp.Context(d, skygen.gaussian_psf(25, 3.0).astype(np.float32), 0.2, **kw)


@pytest.mark.parametrize("shape", [(1, 1), (5, 3), (63, 65), (130, 257)])
@pytest.mark.parametrize("tiles", [0, 1])
@pytest.mark.parametrize("calls", [(1, 2), (31, 1, 1), (32, 33)])
def test_run_is_steps(shape, tiles, calls):
    d = field(*shape)
    a = context(d, threshold=0.0, max_iter=200, max_active=2, peak_tiles=tiles)
    b = context(d, threshold=0.0, max_iter=200, max_active=2, peak_tiles=tiles)
    for n in calls:
        ra = a.run(n)[0]
        rb = 0
        for _ in range(n):
            rb = b.step()
            if rb:
                break
        assert ra == rb
        assert a.counts() == b.counts()
        assert np.array_equal(a.residual(), b.residual())
        assert np.array_equal(a.components_raw(), b.components_raw())
        assert a.residual_sumsq(True) == b.residual_sumsq(True)
    a.close()
    b.close()


@pytest.mark.parametrize("stop", ["threshold", "max_iter"])
def test_run_stops_inside_a_launch(stop):
    d = field(96, 96)
    kw = {"threshold": 0.3, "max_iter": 200} if stop == "threshold" else {"threshold": 0.0, "max_iter": 7}
    a, b = context(d, **kw), context(d, **kw)
    ra, rep = a.run(100)
    rb = 0
    while rb == 0:
        rb = b.step()
    assert ra == rb == (asp.ASP_STOP_THRESHOLD if stop == "threshold" else asp.ASP_STOP_MAXITER)
    assert 0 < rep["iterations"] < 100 and a.counts() == b.counts()
    assert np.array_equal(a.residual(), b.residual())
    assert a.run(5)[0] == ra and a.counts() == b.counts()
    a.close()
    b.close()
