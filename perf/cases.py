"""The work that users of this library have it do, as cases that can be timed.

Every case goes through the package's public calls on synthetic fields made on
the GPU from a seed: a sky of point sources (fluxes dN/dS ~ S^-1.5) and
circular Gaussians, convolved with either a Gaussian PSF or the PSF of a
three-armed array with an earth-rotation track, plus white noise.

Kinds of case
  clean    a dirty image on the GPU to a component list: a context is created,
           the minor cycle runs, the list is read and the residual stays on the
           GPU.  A major cycle of an imager, or the whole of a small job.
  batch    the same for many fields at once (host images, one persistent launch).
  asp2004  the comparison path from a checkpoint: load a state, run iterations.
  refresh  the exact-PSF residual of the present model and its RMS, what a major
           cycle ends with.
  peak     the allocation-free peak search on a caller's image.
  train    Adam steps of the start-value network on recorded pairs.
  forward  the network over many patches (validation of a training run).
"""
import ctypes
import math
import os

import numpy as np
import torch

import paper_1606_07872_amd as asp

C_LIGHT = 299_792_458.0


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def _clean(name, H, W, psf, active, iters, points, gaussians, sigma_hi, **more):
    case = {"kind": "clean", "H": H, "W": W, "psf": psf, "psf_h": 256, "psf_w": 256,
            "active": active, "iters": iters, "points": points, "gaussians": gaussians,
            "sigma_hi": sigma_hi, "gain": 0.1, "noise": 1e-4, "start": "plain", "peak_tiles": 0}
    if name:
        case["name"] = name
    case.update(more)
    return case


def listed():
    return [
        # a small job, where launches and latency count: 128 x 128, Gaussian PSF
        _clean("clean_128", 128, 128, "gauss", 5, 100, 5, 3, 8.0, psf_h=128, psf_w=128,
               noise=1e-3),
        # a facet of odd shape with a cropped, off-centre PSF and a larger active set
        _clean("clean_ragged", 301, 203, "gauss", 8, 60, 20, 8, 20.0, psf_h=91, psf_w=75,
               gain=0.2),
        # an ordinary field
        _clean("clean_1024", 1024, 1024, "array", 5, 100, 200, 40, 40.0),
        # a large mosaic, wide components, an active set of up to ten
        _clean("clean_4096", 4096, 4096, "array", 10, 50, 2000, 300, 120.0),
        # the ordinary field with the learned start values and the incremental
        # peak search
        _clean("clean_learned", 1024, 1024, "array", 5, 60, 200, 40, 40.0, start="learned",
               peak_tiles=1),
        # the ordinary field with the smoothing method's start values
        _clean("clean_smooth", 1024, 1024, "array", 5, 40, 200, 40, 40.0, start="smooth"),
        # a survey: many uneven fields at once
        {"name": "batch_16", "kind": "batch", "fields": 16, "lo": 256, "hi": 1024, "psf": "gauss",
         "psf_h": 64, "psf_w": 64, "active": 5, "iters": 40, "gain": 0.1, "noise": 1e-4},
        # the comparison path of the paper on one facet
        {"name": "asp2004_512", "kind": "asp2004", "H": 512, "W": 512, "psf": "array",
         "psf_h": 256, "psf_w": 256, "iters": 4, "points": 60, "gaussians": 6, "sigma_hi": 12.0,
         "gain": 0.35, "noise": 1e-4},
        # the end of a major cycle on the large mosaic
        {"name": "refresh_4096", "kind": "refresh", "H": 4096, "W": 4096, "psf": "array",
         "psf_h": 256, "psf_w": 256, "model_iters": 40, "points": 2000, "gaussians": 300,
         "sigma_hi": 120.0, "gain": 0.1, "noise": 1e-4},
        # the peak of a caller's own image
        {"name": "peak_4096", "kind": "peak", "H": 4096, "W": 4096},
        # training of the learned start at the trainer's own batch size
        {"name": "train_512", "kind": "train", "rows": 8192, "batch": 512, "steps": 10},
        # validation pass over the pairs of a training run
        {"name": "forward_50000", "kind": "forward", "rows": 50000, "max_batch": 512},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["clean"] * 6 + ["batch", "asp2004", "refresh", "peak", "train", "forward"])
    if kind == "clean":
        H, W = _log_int(rng, 96, 2048), _log_int(rng, 96, 2048)
        area = H * W / 2.0 ** 20
        hi = rng.uniform(4.0, max(6.0, min(H, W) / 16.0))
        psf = rng.choice(["gauss", "array"])
        ph = _log_int(rng, 48, 256)
        return _clean(None, H, W, psf, rng.randint(1, 12), _log_int(rng, 10, 60),
                      max(3, int(200 * area)), max(2, int(40 * area)), round(hi, 2), psf_h=ph,
                      psf_w=min(256, ph + rng.randint(0, 9)), gain=rng.choice([0.05, 0.1, 0.2]),
                      noise=rng.choice([1e-4, 1e-3]),
                      start=rng.choice(["plain", "plain", "learned", "smooth"]),
                      peak_tiles=rng.randint(0, 1))
    if kind == "batch":
        return {"kind": "batch", "fields": rng.randint(2, 16), "lo": _log_int(rng, 100, 256),
                "hi": _log_int(rng, 257, 1024), "psf": "gauss", "psf_h": 64, "psf_w": 64,
                "active": rng.randint(1, 8), "iters": _log_int(rng, 10, 40), "gain": 0.1,
                "noise": 1e-4}
    if kind == "asp2004":
        H, W = _log_int(rng, 128, 512), _log_int(rng, 128, 512)
        return {"kind": "asp2004", "H": H, "W": W, "psf": "array", "psf_h": 128, "psf_w": 128,
                "iters": rng.randint(2, 4), "points": 40, "gaussians": 5,
                "sigma_hi": round(rng.uniform(3.0, 12.0), 2), "gain": 0.35, "noise": 1e-4}
    if kind == "refresh":
        H, W = _log_int(rng, 256, 4096), _log_int(rng, 256, 4096)
        area = H * W / 2.0 ** 20
        return {"kind": "refresh", "H": H, "W": W, "psf": "array", "psf_h": 256, "psf_w": 256,
                "model_iters": rng.randint(20, 40), "points": max(10, int(120 * area)),
                "gaussians": max(3, int(19 * area)), "sigma_hi": round(min(H, W) / 34.0 + 4.0, 2),
                "gain": 0.1, "noise": 1e-4}
    if kind == "peak":
        return {"kind": "peak", "H": _log_int(rng, 100, 5000), "W": _log_int(rng, 100, 5000)}
    if kind == "train":
        return {"kind": "train", "rows": 8192, "batch": _log_int(rng, 32, 1024),
                "steps": rng.randint(4, 10)}
    return {"kind": "forward", "rows": _log_int(rng, 500, 50000),
            "max_batch": rng.choice([256, 512, 1024])}


# ---------------------------------------------------------------------------
# Synthetic fields
# ---------------------------------------------------------------------------

def _gauss_psf(Hp, Wp, fwhm, cy, cx, device):
    sig = fwhm / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    r = torch.arange(Hp, dtype=torch.float64, device=device) - cy
    c = torch.arange(Wp, dtype=torch.float64, device=device) - cx
    return torch.exp(-(r[:, None] ** 2 + c[None, :] ** 2) / (2.0 * sig * sig))


def _smooth_even(n):
    """The least even size >= n with no prime factor above 7."""
    m = n + n % 2
    while True:
        r = m
        for f in (2, 3, 5, 7):
            while r % f == 0:
                r //= f
        if r == 1:
            return m
        m += 2


def _array_grid(g, device):
    """Uniformly weighted, tapered uv sampling of a 27-antenna Y array over an
    eight-hour track and 32 channels of 1..2 GHz, on a g x g grid (FFT layout)."""
    k = torch.arange(1, 10, dtype=torch.float64, device=device)
    arm = 5200.0 * (k / 9.0) ** 1.716
    az = torch.tensor([5.0, 125.0, 245.0], dtype=torch.float64, device=device) * math.pi / 180.0
    east = (arm[None, :] * torch.sin(az)[:, None]).reshape(-1)
    north = (arm[None, :] * torch.cos(az)[:, None]).reshape(-1)
    lat, dec = math.radians(34.0), math.radians(40.0)
    i, j = torch.triu_indices(27, 27, 1, device=device)
    bx = -math.sin(lat) * (north[j] - north[i])
    by = east[j] - east[i]
    bz = math.cos(lat) * (north[j] - north[i])
    ha = torch.linspace(-4.0, 4.0, 481, dtype=torch.float64, device=device) * (math.pi / 12.0)
    sh, ch = torch.sin(ha)[:, None], torch.cos(ha)[:, None]
    u = sh * bx + ch * by
    v = -math.sin(dec) * ch * bx + math.sin(dec) * sh * by + math.cos(dec) * bz
    lam = (1e9 + (torch.arange(32, dtype=torch.float64, device=device) + 0.5) * (1e9 / 32)) / C_LIGHT
    u = (u.reshape(-1, 1) * lam).reshape(-1)
    v = (v.reshape(-1, 1) * lam).reshape(-1)
    du = float(torch.maximum(u.abs().max(), v.abs().max())) / (0.30 * g)
    iu, iv = torch.round(u / du).long(), torch.round(v / du).long()
    grid = torch.zeros(g * g, dtype=torch.float64, device=device)
    grid[(iv % g) * g + iu % g] = 1.0
    grid[(-iv % g) * g + (-iu) % g] = 1.0
    f = torch.fft.fftfreq(g, dtype=torch.float64, device=device) * g
    tap = torch.exp(-f * f / (2.0 * (0.45 * 0.30 * g) ** 2))
    return grid.reshape(g, g) * tap[:, None] * tap[None, :]


def _sky(gen, H, W, points, gaussians, sigma_hi, device):
    def uniform(n, lo, hi):
        return lo + (hi - lo) * torch.rand(n, generator=gen, dtype=torch.float64)

    e = min(8, (min(H, W) - 1) // 4)
    px = uniform(points, e, W - e).floor().long()
    py = uniform(points, e, H - e).floor().long()
    a, b = 1e-3 ** -0.5, 1.0
    flux = (a + uniform(points, 0.0, 1.0) * (b - a)) ** -2.0
    sky = torch.zeros(H, W, dtype=torch.float64, device=device)
    sky.index_put_((py.to(device), px.to(device)), flux.to(device), accumulate=True)
    for _ in range(gaussians):
        sig = float(uniform(1, 2.0, sigma_hi))
        m = min(3.0 * sig, 0.45 * min(H, W))
        x, y = float(uniform(1, m, W - 1 - m)), float(uniform(1, m, H - 1 - m))
        peak, h = float(uniform(1, 0.05, 0.5)), math.ceil(8.0 * sig)
        r0, r1 = max(0, int(y) - h), min(H, int(y) + h + 2)
        c0, c1 = max(0, int(x) - h), min(W, int(x) + h + 2)
        r = torch.arange(r0, r1, dtype=torch.float64, device=device) - y
        c = torch.arange(c0, c1, dtype=torch.float64, device=device) - x
        sky[r0:r1, c0:c1] += peak * torch.exp(-r * r / (2 * sig * sig))[:, None] \
            * torch.exp(-c * c / (2 * sig * sig))[None, :]
    return sky


def _field(case, seed, device="cuda"):
    """(dirty, psf): float32 images on the device."""
    H, W, Hp, Wp = case["H"], case["W"], case["psf_h"], case["psf_w"]
    gen = torch.Generator().manual_seed(int(seed))
    g = _smooth_even(max(H + Hp, W + Wp, 2 * max(H, W)))
    sky = _sky(gen, H, W, case["points"], case["gaussians"], case["sigma_hi"], device)
    # the PSF's peak pixel: the centre, or a little off it when the crop is odd
    cy, cx = Hp // 2 - (3 if Hp % 2 else 0), Wp // 2 + (2 if Wp % 2 else 0)
    if case["psf"] == "gauss":
        fwhm = 3.0 if H <= 128 else 2.5 + 3.5 * float(torch.rand(1, generator=gen))
        psf = _gauss_psf(Hp, Wp, fwhm, cy, cx, device)
        whole = torch.zeros(g, g, dtype=torch.float64, device=device)
        whole[:Hp, :Wp] = psf
        spec = torch.fft.rfft2(torch.roll(whole, (-cy, -cx), (0, 1)))
    else:
        grid = _array_grid(g, device)
        whole = torch.fft.ifft2(grid).real
        norm = float(whole[0, 0])
        psf = torch.roll(whole, (cy, cx), (0, 1))[:Hp, :Wp] / norm
        spec = (grid[:, : g // 2 + 1] / norm).to(torch.complex128)
    dirty = torch.fft.irfft2(torch.fft.rfft2(sky, s=(g, g)) * spec, s=(g, g))[:H, :W]
    noise = torch.randn(H, W, generator=torch.Generator(device).manual_seed(int(seed) + 1),
                        dtype=torch.float64, device=device)
    dirty = dirty + case["noise"] * noise
    return dirty.float().contiguous(), psf.float().contiguous()


class _DeviceImage:
    """A context's residual for torch.as_tensor, without a copy."""

    def __init__(self, ctx):
        self.ctx = ctx
        self.__cuda_array_interface__ = {"shape": (ctx.H, ctx.W), "typestr": "<f4", "version": 2,
                                         "data": (ctx.residual_device_ptr(), False)}


def _residual(ctx):
    """The residual as a tensor that keeps its context alive: the context's memory is
    given back when the last output of a pass is dropped."""
    view = torch.as_tensor(_DeviceImage(ctx), device="cuda")
    view.ctx = ctx
    return view


def _components(ctx, rows):
    """The fitted list (a, x, y, s), zeros after its end: an iteration whose new
    component has amplitude zero adds no row."""
    out = np.zeros((rows, 4))
    got = ctx.components_raw()
    out[:len(got)] = got
    return out


def _weights(seed):
    """He-uniform weights in the flat order of the network, zero biases."""
    rng = np.random.default_rng(seed)
    parts, dims = [], (asp.MLP_IN, 256, 256, asp.MLP_OUT)
    for i in range(3):
        lim = math.sqrt((6.0 if i < 2 else 3.0) / dims[i])
        parts += [rng.uniform(-lim, lim, dims[i + 1] * dims[i]), np.zeros(dims[i + 1])]
    return np.concatenate(parts).astype(np.float32)


def _pairs(rows, seed):
    """Patches as the minor cycle records them (a Gaussian near the middle of 32 x
    32 pixels, peak 1, a second source and noise) and their targets."""
    gen = torch.Generator("cuda").manual_seed(int(seed))

    def uniform(lo, hi):
        return lo + (hi - lo) * torch.rand(rows, 1, 1, generator=gen, device="cuda")

    p = torch.arange(32, device="cuda", dtype=torch.float32) - 16.0
    s, dx, dy, amp = uniform(1.3, 9.0), uniform(-1, 1), uniform(-1, 1), uniform(0.8, 1.2)
    ex, ey, es, ea = uniform(-14, 14), uniform(-14, 14), uniform(1.3, 5.0), uniform(-0.3, 0.5)
    img = amp * torch.exp(-((p[None, None, :] - dx) ** 2 + (p[None, :, None] - dy) ** 2) / (2 * s * s))
    img = img + ea * torch.exp(-((p[None, None, :] - ex) ** 2 + (p[None, :, None] - ey) ** 2)
                               / (2 * es * es))
    img = img + 0.01 * torch.randn(img.shape, generator=gen, device="cuda")
    x = img.reshape(rows, asp.MLP_IN).contiguous()
    t = torch.stack([amp, torch.log(s / 1.3), dx, dy], 1).reshape(rows, asp.MLP_OUT).contiguous()
    return x, t


# ---------------------------------------------------------------------------
# What a program has in hand, one pass, and its least work
# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "clean":
        s["dirty"], s["psf"] = _field(case, seed)
        if case["start"] == "learned":
            s["weights"] = np.load(os.path.join(os.path.dirname(asp.__file__),
                                                "proposal_weights.npy"))
    elif kind == "batch":
        rng = np.random.default_rng(seed)
        s["fields"] = []
        for i in range(case["fields"]):
            # the sizes belong to the case, so that every seed costs about the same
            n = int(round(case["lo"] * (case["hi"] / case["lo"]) ** (i / max(1, case["fields"] - 1))))
            area = n * n / 2.0 ** 20
            one = dict(case, H=n, W=n, points=max(2, int(200 * area)),
                       gaussians=max(1, int(40 * area)), sigma_hi=max(3.0, min(40.0, n / 16.0)))
            d, p = _field(one, int(rng.integers(1 << 31)))
            s["fields"].append((d.cpu().numpy(), p.cpu().numpy(), case["gain"], 0.0))
    elif kind == "asp2004":
        d, p = _field(case, seed)
        torch.cuda.synchronize()
        s["ctx"] = asp.Context(d, p, case["gain"], 0.0, max_iter=100, smooth_norm=1)
        s["blob"] = s["ctx"].save_state()
        s["ctx"].run_2004(1)                 # buffers and FFT plans of a running program
    elif kind == "refresh":
        d, p = _field(case, seed)
        torch.cuda.synchronize()
        s["ctx"] = asp.Context(d, p, case["gain"], 0.0, max_iter=case["model_iters"], max_active=5)
        s["dirty"], s["psf"] = d, p
        s["ctx"].run(case["model_iters"])
        s["ctx"].refresh_residual()          # buffers and FFT plans of a running program
    elif kind == "peak":
        gen = torch.Generator("cuda").manual_seed(int(seed))
        s["image"] = torch.randn(case["H"], case["W"], generator=gen, device="cuda")
        s["idx"] = torch.zeros(1, dtype=torch.int64, device="cuda")
        s["value"] = torch.zeros(1, dtype=torch.float32, device="cuda")
    elif kind == "train":
        s["x"], s["t"] = _pairs(case["rows"], seed)
        order = np.random.default_rng(seed).integers(0, case["rows"], case["steps"] * case["batch"])
        s["order"] = torch.from_numpy(order.astype(np.int32)).cuda()
        s["net"] = asp.Mlp(_weights(seed), max_batch=case["batch"])
    else:
        s["x"], _ = _pairs(case["rows"], seed)
        s["y"] = torch.empty(case["rows"], asp.MLP_OUT, device="cuda")
        s["net"] = asp.Mlp(_weights(seed), max_batch=case["max_batch"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "clean":
        ctx = asp.Context(s["dirty"], s["psf"], case["gain"], 0.0, max_iter=case["iters"],
                          max_active=case["active"], peak_tiles=case["peak_tiles"],
                          init_mode=2 if case["start"] == "smooth" else 0)
        if case["start"] == "learned":
            ctx.set_mlp(s["weights"])
            ctx.set_init_mode(1)
        ctx.run(case["iters"])
        return {"components": _components(ctx, case["iters"]), "residual": _residual(ctx)}
    if kind == "batch":
        b = asp.Batch(s["fields"], max_iter=case["iters"], max_active=case["active"])
        b.run(case["iters"])
        views = [b.field(i) for i in range(b.n)]
        return {"components": [_components(v, case["iters"]) for v in views],
                "residuals": [_residual(v) for v in views]}
    if kind == "asp2004":
        s["ctx"].load_state(s["blob"])
        s["ctx"].run_2004(case["iters"])
        return {"components": _components(s["ctx"], case["iters"]), "residual": _residual(s["ctx"])}
    if kind == "refresh":
        s["ctx"].refresh_residual()
        return {"rms": s["ctx"].residual_rms(), "residual": _residual(s["ctx"])}
    if kind == "peak":
        img = s["image"]
        rc = asp.lib().asp_find_peak_noalloc(
            img.data_ptr(), img.shape[0], img.shape[1], s["idx"].data_ptr(), s["value"].data_ptr(),
            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        if rc != asp.ASP_OK:
            raise asp.AspError(rc, "asp_find_peak_noalloc")
        return {"idx": s["idx"], "value": s["value"]}
    if kind == "train":
        loss = s["net"].train(s["x"], s["t"], s["order"], case["batch"])
        return {"loss": loss, "weights": s["net"].weights()}
    s["net"].forward(s["x"], s["y"])
    return s["y"]


def work(case):
    """Each input read once and each output written once; the multiply-adds of the
    network's products; of the FFT convolutions the transforms' usual count."""
    kind = case["kind"]
    if kind == "batch":
        n = [case["lo"] * (case["hi"] / case["lo"]) ** (i / max(1, case["fields"] - 1))
             for i in range(case["fields"])]
        return {"bytes": sum(8.0 * v * v for v in n), "flops": 0.0}
    if kind in ("clean", "asp2004", "refresh"):
        H, W, Hp, Wp = case["H"], case["W"], case["psf_h"], case["psf_w"]
        flops = 0.0
        if kind == "refresh":
            n = (H + Hp - 1.0) * (W + Wp - 1.0)
            flops = 2 * 2.5 * n * math.log2(n) + 3 * n
        return {"bytes": 8.0 * H * W + 4.0 * Hp * Wp, "flops": flops}
    if kind == "peak":
        return {"bytes": 4.0 * case["H"] * case["W"] + 12, "flops": 0.0}
    macs = asp.MLP_IN * 256 + 256 * 256 + 256 * asp.MLP_OUT
    if kind == "train":
        rows = case["batch"] * case["steps"]
        # backward: the weights' gradients, and the inputs' of layers 2 and 3
        return {"bytes": 4.0 * rows * (asp.MLP_IN + asp.MLP_OUT + 1) + 8.0 * asp.MLP_PARAMS,
                "flops": 2.0 * rows * (3 * macs - asp.MLP_IN * 256)}
    return {"bytes": 4.0 * case["rows"] * (asp.MLP_IN + asp.MLP_OUT) + 4.0 * asp.MLP_PARAMS,
            "flops": 2.0 * case["rows"] * macs}


# ---------------------------------------------------------------------------
# The same in 64 bits, by plain torch
# ---------------------------------------------------------------------------

def _unpack(w):
    w = torch.as_tensor(w).cuda().double()
    out, at = [], 0
    for n, k in ((256, asp.MLP_IN), (256, 256), (asp.MLP_OUT, 256)):
        out.append(w[at:at + n * k].reshape(n, k).contiguous())
        out.append(w[at + n * k:at + n * k + n].contiguous())
        at += n * k + n
    return out


def _exact_train(case, seed):
    x, t = _pairs(case["rows"], seed)
    x, t = x.double(), t.double()
    order = np.random.default_rng(seed).integers(0, case["rows"], case["steps"] * case["batch"])
    order = torch.from_numpy(order).cuda().reshape(case["steps"], case["batch"])
    P = [p.clone() for p in _unpack(_weights(seed))]
    m, v = [torch.zeros_like(p) for p in P], [torch.zeros_like(p) for p in P]
    total = 0.0
    for k in range(case["steps"]):
        X, T = x[order[k]], t[order[k]]
        z1 = X @ P[0].T + P[1]
        h1 = z1.clamp(min=0)
        z2 = h1 @ P[2].T + P[3]
        h2 = z2.clamp(min=0)
        d = h2 @ P[4].T + P[5] - T
        total += float((d * d).mean())
        dy = 2.0 * d / d.numel()
        d2 = (dy @ P[4]) * (z2 > 0)
        d1 = (d2 @ P[2]) * (z1 > 0)
        grads = [d1.T @ X, d1.sum(0), d2.T @ h1, d2.sum(0), dy.T @ h2, dy.sum(0)]
        for p, g, mi, vi in zip(P, grads, m, v):
            mi.mul_(0.9).add_(0.1 * g)
            vi.mul_(0.999).add_(0.001 * g * g)
            p -= 1e-3 * (mi / (1 - 0.9 ** (k + 1))) / (torch.sqrt(vi / (1 - 0.999 ** (k + 1))) + 1e-8)
    return {"loss": total / case["steps"],
            "weights": torch.cat([p.reshape(-1) for p in P]).cpu().numpy()}


def _lanczos3(u):
    return torch.where(u.abs() < 3.0, torch.sinc(u) * torch.sinc(u / 3.0), torch.zeros_like(u))


def _model(ctx, H, W):
    """The components of a context's list in the sky plane, rendered in 64 bits: at
    least 1 px wide as sampled Gaussians on the window of 5 widths, narrower ones by
    three Gauss-Hermite nodes per axis spread with Lanczos-3."""
    ab, wb = ctx.psf_gauss()
    img = torch.zeros(H, W, dtype=torch.float64, device="cuda")
    for a, x, y, s in ctx.components_raw():
        flux = a * s * s / (ab * wb * wb)
        om = math.sqrt(max(s * s - wb * wb, 0.0))
        axes = []
        for ctr, n in ((y, H), (x, W)):
            if om >= 1.0:
                h = max(3, math.ceil(5.0 * om))
                p = torch.arange(math.floor(ctr + 0.5) - h, math.floor(ctr + 0.5) + h + 1, device="cuda")
                w = torch.exp(-(p.double() - ctr) ** 2 / (2.0 * om * om))
            else:
                d = math.sqrt(3.0) * (om if om > 1e-6 * wb else 0.0)
                p = torch.arange(math.floor(ctr) - 5, math.floor(ctr) + 7, device="cuda")
                u = p.double() - ctr
                w = 2.0 / 3.0 * _lanczos3(u) + (_lanczos3(u - d) + _lanczos3(u + d)) / 6.0
                w = w / w.sum()
            keep = (p >= 0) & (p < n)
            axes.append((p[keep], w[keep]))
        (pr, wr), (pc, wc) = axes
        if len(pr) and len(pc):
            scale = flux / (2.0 * math.pi * om * om) if om >= 1.0 else flux
            img[int(pr[0]):int(pr[-1]) + 1, int(pc[0]):int(pc[-1]) + 1] += scale * wr[:, None] * wc[None, :]
    return img


def exact(case, seed):
    kind = case["kind"]
    if kind == "peak":
        s = prepare(case, seed)
        a = s["image"].double().reshape(-1)
        top = (a.abs() == a.abs().max()).nonzero()[:1, 0]
        return {"idx": top, "value": a[top]}
    if kind == "refresh":
        # the model is an input of this path: the list as prepare() left it
        s = prepare(case, seed)
        H, W = case["H"], case["W"]
        Hp, Wp = s["psf"].shape
        gh, gw = _smooth_even(H + Hp - 1), _smooth_even(W + Wp - 1)
        at = int(s["psf"].argmax())
        full = torch.fft.irfft2(torch.fft.rfft2(_model(s["ctx"], H, W), s=(gh, gw))
                                * torch.fft.rfft2(s["psf"].double(), s=(gh, gw)), s=(gh, gw))
        ci, cj = at // Wp, at % Wp
        r = s["dirty"].double() - full[ci:ci + H, cj:cj + W]
        return {"rms": math.sqrt(float((r * r).mean())), "residual": r}
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "forward":
        x, _ = _pairs(case["rows"], seed)
        w1, b1, w2, b2, w3, b3 = _unpack(_weights(seed))
        h = (x.double() @ w1.T + b1).clamp(min=0)
        return (h @ w2.T + b2).clamp(min=0) @ w3.T + b3
    return None          # a fit's end has no closed form: the iterations are the definition
