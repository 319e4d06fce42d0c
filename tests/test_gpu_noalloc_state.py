"""The allocation-free peak search answers from its own image alone: after a call
whose second kernel never ran, and after an image of NaN, which has no peak."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
asp = pytest.importorskip("paper_1606_07872_amd")


class Search:
    def __init__(self):
        self.stream = torch.cuda.Stream()
        self.idx = torch.full((1,), -1, dtype=torch.int64, device="cuda")
        self.val = torch.zeros((1,), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()

    def enqueue(self, R):
        H, W = R.shape
        return asp.lib().asp_find_peak_noalloc(R.data_ptr(), H, W, self.idx.data_ptr(),
                                               self.val.data_ptr(), self.stream.cuda_stream)

    def __call__(self, R):
        torch.cuda.synchronize()
        assert self.enqueue(R) == asp.ASP_OK
        self.stream.synchronize()
        return int(self.idx.item()), float(self.val.item())


def image(H, W, scale):
    rng = np.random.default_rng(H * W)
    return (scale * rng.normal(0.0, 1.0, size=(H, W))).astype(np.float32)


def expect(img):
    i = int(np.argmax(np.abs(img.ravel())))
    return i, float(img.ravel()[i])


SHAPES = [(1, 1), (1, 3), (33, 31), (511, 4097), (1500, 2001)]


@pytest.mark.parametrize("shape", SHAPES)
def test_image_of_nan(shape):
    s = Search()
    nan = torch.full(shape, float("nan"), dtype=torch.float32, device="cuda")
    idx, val = s(nan)
    assert idx == 2 ** 32 - 1 and np.isnan(val)
    img = image(*shape, 1.0)
    assert s(torch.from_numpy(img).cuda()) == expect(img)
    # NaN among numbers is passed over; an infinity is the peak
    img.ravel()[0] = np.nan
    if img.size > 1:
        img.ravel()[-1] = -np.inf
        assert s(torch.from_numpy(img).cuda()) == (img.size - 1, -np.inf)


def test_after_a_scan_without_an_answer():
    """The first kernel of a large image's search, captured and launched without
    the second, then searches of smaller and fainter images."""
    hip = ctypes.CDLL("libamdhip64.so.7")

    def call(name, *args):
        rc = getattr(hip, name)(*args)
        assert rc == 0, (name, rc)

    vp = ctypes.c_void_p
    s = Search()
    big = torch.from_numpy(image(2000, 2100, 50.0)).cuda()
    s(big)                                  # the scratch's address is known before the capture
    st = vp(s.stream.cuda_stream)
    graph, ex = vp(), vp()
    call("hipStreamBeginCapture", st, 1)
    rc = s.enqueue(big)
    call("hipStreamEndCapture", st, ctypes.byref(graph))
    assert rc == asp.ASP_OK
    n = ctypes.c_size_t(0)
    call("hipGraphGetNodes", graph, None, ctypes.byref(n))
    assert n.value == 2
    nodes, root, one = (vp * 2)(), (vp * 1)(), ctypes.c_size_t(1)
    call("hipGraphGetNodes", graph, nodes, ctypes.byref(n))
    call("hipGraphGetRootNodes", graph, root, ctypes.byref(one))
    assert one.value == 1
    for node in nodes:
        if node != root[0]:
            call("hipGraphDestroyNode", vp(node))
    call("hipGraphInstantiate", ctypes.byref(ex), graph, None, None, ctypes.c_size_t(0))
    for shape in SHAPES + [(2000, 2100)]:
        call("hipGraphLaunch", ex, st)
        s.stream.synchronize()
        img = image(*shape, 1.0)
        assert s(torch.from_numpy(img).cuda()) == expect(img)
    call("hipGraphExecDestroy", ex)
    call("hipGraphDestroy", graph)
