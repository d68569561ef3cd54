"""Workloads of the sliding-window correlation as a program calls it: single
images of every element type, batches, volumes, series, the cloud filter and
runs from host memory.

    listed()            the workloads that stand for each kind of use
    draw(rng)           one more workload of the same ranges
    prepare(case, seed) inputs on the GPU, and the plan a program would keep
    run(state)          one pass through the public entry points
    work(case)          bytes and operations one pass cannot do without
    exact(case, seed)   the same outputs from plain torch in 64 bits

Shapes, windows and steps are texts such as "768x1024" (numpy order, the last
axis contiguous).
"""
import math

import torch

import paper_1807_06507_amd as swc

DTYPES = {"u8": torch.uint8, "u16": torch.uint16, "f32": torch.float32}
ITEM = {"u8": 1, "u16": 2, "f32": 4}
INVALID = -2.0
MISSING = -999.0


def _image(name, shape, dtype, window, step="1x1", border="clip", flags=False, missing=0.0,
           scene="cloud"):
    c = dict(kind="image", shape=shape, dtype=dtype, window=window, step=step, border=border,
             flags=flags, missing=missing, scene=scene)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a crop around one detection: the call itself is the cost
        _image("crop_f32_96x128_k7", "96x128", "f32", "7x7", border="fill", flags=True),
        # one scene of cloud reflectances, float
        _image("image_f32_768x1024_k7", "768x1024", "f32", "7x7"),
        # the night-light pair of the paper's size class (visible and infrared counts)
        _image("image_u16_3000x4000_k7", "3000x4000", "u16", "7x7", border="fill", scene="night"),
        # a large offset pair under a wide window (the precision sweep's image)
        _image("image_f32_4096x4096_k15", "4096x4096", "f32", "15x15", scene="offset"),
        # 8-bit quick-look of a swath whose rows are no multiple of anything
        _image("swath_u8_2161x3239_k11", "2161x3239", "u8", "11x11", flags=True, scene="night"),
        # reprojected float scene with data gaps, rectangular window, thinned output
        _image("gaps_f32_1531x2047_k13x21_s2", "1531x2047", "f32", "13x21", step="2x2",
               border="valid", flags=True, missing=2e-4),
        # an archive of scenes of mixed size and window in one plan
        dict(kind="batch", name="batch_f32_16", pairs=16, dtype="f32", sizes=1, min_side=256,
             max_side=4096, flags=False),
        # a dense volume, cubic window
        dict(kind="volume", name="volume_f32_256x512x512_k7", shape="256x512x512", dtype="f32",
             window="7x7x7", step="1x1x1", border="clip", flags=False, missing=0.0),
        # an image stack in time: odd sides, shallow window
        dict(kind="volume", name="stack_u16_61x187x301_k3x5x7", shape="61x187x301", dtype="u16",
             window="3x5x7", step="1x1x1", border="fill", flags=True, missing=0.0),
        # a long pair of series, wide window
        dict(kind="series", name="series_f32_2p28_k1001", shape=str(1 << 28), dtype="f32",
             window="1001", step="1", border="clip", flags=False, missing=0.0),
        # the application: map, cloud mask, filter of the light detections
        dict(kind="filter", name="filter_u16_1536x2048_k7", shape="1536x2048", window="7x7",
             detections=4000, tau=0.5),
        # host memory to host memory (the paper's timing includes the transfers)
        dict(kind="host", name="host_u16_3000x4000_k7", shape="3000x4000", dtype="u16",
             window="7x7", border="fill", band=512, depth=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _sides(rng, lo, hi, most):
    """Two sides spread over their logarithm; a product above `most` is cut."""
    h, w = _log(rng, lo, hi), _log(rng, lo, hi)
    if h * w > most:
        h = max(lo, int(most // w))
    return h, w


def draw(rng):
    """One more workload of the ranges the listed ones stand for."""
    kind = rng.choice(["image"] * 5 + ["batch", "volume", "volume", "series", "series", "filter",
                                       "host"])
    dtype = rng.choice(["u8", "u16", "f32"])
    border = rng.choice(["fill", "clip", "clip", "valid"])
    flags = rng.random() < 0.4
    if kind == "image":
        if rng.random() < 0.6:
            k = rng.choice([3, 5, 7, 9, 15, 31])
            kh, kw, most = k, k, 1 << 24
        else:
            kh, kw, most = rng.randint(2, 31), rng.randint(2, 31), 1 << 22
        h, w = _sides(rng, 48, 4096, most)
        s = rng.choice([1, 1, 1, 1, 2, 3, 4])
        return _image(None, "%dx%d" % (h, w), dtype, "%dx%d" % (kh, kw), "%dx%d" % (s, s), border,
                      flags, rng.choice([0.0, 0.0, 2e-4]) if dtype == "f32" else 0.0,
                      rng.choice(["cloud", "offset"]) if dtype == "f32" else "night")
    if kind == "batch":
        lo = _log(rng, 64, 512)
        return dict(kind="batch", pairs=rng.randint(3, 16), dtype=rng.choice(["f32", "f32", "u16"]),
                    sizes=rng.randint(0, 1 << 20), min_side=lo, max_side=_log(rng, lo, 3000),
                    flags=flags)
    if kind == "volume":
        d = _log(rng, 12, 200)
        h, w = _sides(rng, 32, 500, (1 << 23) // d)
        kx = rng.choice([3, 5, 7, 9])
        kz, ky = (kx, kx) if rng.random() < 0.5 else (rng.randint(2, 9), rng.randint(2, 9))
        s = rng.choice([1, 1, 1, 2])
        return dict(kind="volume", shape="%dx%dx%d" % (d, h, w), dtype=dtype,
                    window="%dx%dx%d" % (kz, ky, kx), step="%dx%dx%d" % (s, s, s), border=border,
                    flags=flags, missing=rng.choice([0.0, 0.0, 2e-4]) if dtype == "f32" else 0.0)
    if kind == "series":
        return dict(kind="series", shape=str(_log(rng, 4000, 1 << 26)), dtype=dtype,
                    window=str(_log(rng, 3, 1448)), step=str(rng.choice([1, 1, 1, 5])),
                    border=border, flags=flags,
                    missing=rng.choice([0.0, 0.0, 2e-5]) if dtype == "f32" else 0.0)
    if kind == "filter":
        h, w = _sides(rng, 200, 3000, 1 << 23)
        return dict(kind="filter", shape="%dx%d" % (h, w), window=rng.choice(["5x5", "7x7", "9x9"]),
                    detections=_log(rng, 100, 20000), tau=0.5)
    h, w = _sides(rng, 300, 4000, 12000000)
    return dict(kind="host", shape="%dx%d" % (h, w), dtype=rng.choice(["u16", "f32"]),
                window=rng.choice(["5x5", "7x7", "9x9"]), border=rng.choice(["fill", "clip"]),
                band=rng.choice([256, 512]), depth=3)


# ---- inputs -----------------------------------------------------------------

def _ints(text):
    return tuple(int(v) for v in text.split("x"))


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, shape, mean=0.0, std=1.0):
    return torch.randn(shape, generator=g, device="cuda").mul_(std).add_(mean)


def _unit(g, shape):
    return torch.rand(shape, generator=g, device="cuda")


def _coarse_mask(g, h, w, cover):
    """Smooth noise above its quantile: patches some 40 pixels across."""
    n = torch.randn((1, 1, h // 40 + 2, w // 40 + 2), generator=g, device="cuda")
    f = torch.nn.functional.interpolate(n, size=(h, w), mode="bicubic", align_corners=True)[0, 0]
    return f > 1.0 - 2.0 * cover


def _cloud(g, h, w):
    """Lognormal reflectances, anti-correlated under the clouds."""
    x = _normal(g, (h, w)).exp_()
    y = torch.where(_coarse_mask(g, h, w, 0.3), -0.6 * x + _normal(g, (h, w), 0.0, 0.5),
                    _normal(g, (h, w)).exp_())
    return x, y


def _offset(g, h, w):
    """A large mean with unit variance; the correlation differs by block."""
    x = _normal(g, (h, w), 1000.0, 1.0)
    rho = _unit(g, (h // 64 + 1, w // 64 + 1)).mul_(2.0).sub_(1.0)
    rho = rho.repeat_interleave(64, 0).repeat_interleave(64, 1)[:h, :w]
    return x, rho * x + _normal(g, (h, w)) * torch.sqrt(1.0 - rho * rho)


def _night(g, h, w, bits):
    """Visible counts with point lights and moonlit clouds, infrared counts
    that are lower over the clouds.  Returns the pair and the lights' places."""
    top = float((1 << bits) - 1)
    unit = 200.0 if bits == 16 else 40.0
    vis = torch.poisson(torch.full((h, w), unit, device="cuda"), generator=g)
    n = max(1, h * w // 10000)
    at = torch.randint(0, h * w, (n,), generator=g, device="cuda")
    vis.view(-1)[at] = _unit(g, (n,)).mul_(0.6 * top).add_(0.3 * top)
    m = _coarse_mask(g, h, w, 0.3).float()
    ir = _normal(g, (h, w), 0.46 * top, 0.0122 * top + 0.5)
    ir -= m * _unit(g, (h, w)).mul_(0.06 * top).add_(0.03 * top)
    vis += m * _unit(g, (h, w)).mul_(0.1 * top).add_(0.015 * top)
    cast = torch.uint8 if bits == 8 else torch.int32
    x, y = (v.round_().clamp_(0, top).to(cast) for v in (vis, ir))
    if bits == 16:
        x, y = x.to(torch.uint16), y.to(torch.uint16)
    return x, y, at


def _gaps(g, x, y, share):
    """Missing values: single cells in both arrays and a few runs of cells."""
    for a in (x, y):
        flat = a.view(-1)
        n = max(1, int(flat.numel() * share))
        flat[torch.randint(0, flat.numel(), (n,), generator=g, device="cuda")] = MISSING
    starts = torch.randint(0, max(1, x.numel() - 40), (4,), generator=g, device="cuda")
    at = (starts[:, None] + torch.arange(40, device="cuda")[None, :]).view(-1)
    x.view(-1)[at.clamp_(max=x.numel() - 1)] = MISSING


def _image_pair(case, g, h, w):
    if case["dtype"] == "u8":
        return _night(g, h, w, 8)[:2]
    if case["dtype"] == "u16":
        return _night(g, h, w, 16)[:2]
    x, y = (_offset if case.get("scene") == "offset" else _cloud)(g, h, w)
    x, y = x.contiguous(), y.contiguous()
    if case.get("missing"):
        _gaps(g, x, y, case["missing"])
    return x, y


def _quantise(case, x, y, scale):
    """A float pair as the case's type (integers around the middle of the range)."""
    if case["dtype"] == "f32":
        return x.contiguous(), y.contiguous()
    top = 255.0 if case["dtype"] == "u8" else 65535.0
    return tuple((v * (scale * top)).add_(0.5 * top).round_().clamp_(0, top).to(torch.int32)
                 .to(DTYPES[case["dtype"]]) for v in (x, y))


def _volume_pair(case, g, shape):
    """A smooth field of unit deviation and a noisy anti-correlated one."""
    x = _normal(g, shape)
    for d in range(3):
        if shape[d] > 4:
            x = (x + x.roll(1, d) + x.roll(-1, d) + x.roll(2, d) + x.roll(-2, d)).div_(5 ** 0.5)
    y = -0.8 * x + _normal(g, shape, 0.0, 0.6)
    return _quantise(case, x, y, 0.1)


def _series_pair(case, g, n):
    """Two first-order autoregressive series with correlated innovations."""
    e, f = _normal(g, (n,)), _normal(g, (n,))
    f.mul_(0.75 ** 0.5).add_(e, alpha=0.5)
    for v in (e, f):
        for k in range(8):
            lag = 1 << k
            if lag < n:
                v[lag:] += v[:-lag].clone().mul_(0.95 ** lag)
    return _quantise(case, e, f, 0.06)


def _batch_shapes(case):
    import random
    r = random.Random(case["sizes"])
    lo, hi = case["min_side"], case["max_side"]
    return [(r.randint(lo, max(lo, hi * 3 // 4)), r.randint(lo, hi), r.choice([5, 7, 9, 15]))
            for _ in range(case["pairs"])]


def _inputs(case, seed):
    """The pair, or the list of pairs, that a pass reads."""
    g = _gen(seed)
    if case["kind"] == "batch":
        return [_image_pair(case, g, h, w) for h, w, _ in _batch_shapes(case)]
    shape = _ints(case["shape"])
    if case["kind"] == "volume":
        x, y = _volume_pair(case, g, shape)
    elif case["kind"] == "series":
        x, y = _series_pair(case, g, shape[0])
    elif case["kind"] == "filter":
        return _night(g, shape[0], shape[1], 16)
    else:
        return _image_pair(case, g, *shape)
    if case["missing"]:
        _gaps(g, x, y, case["missing"])
    return x, y


def prepare(case, seed):
    got = _inputs(case, seed)
    state = dict(case=case)
    if case["kind"] == "batch":
        pairs = [dict(x=x, y=y, window=(k, k), step=1, border="clip")
                 for (x, y), (_, _, k) in zip(got, _batch_shapes(case))]
        state["plan"] = swc.BatchPlan(pairs, return_flags=case["flags"])
    elif case["kind"] == "filter":
        state["x"], state["y"], lights = got
        state["idx"] = lights[torch.randint(0, lights.numel(), (case["detections"],),
                                            generator=_gen(seed + 1), device="cuda")]
    elif case["kind"] == "host":
        state["x"], state["y"] = (v.cpu().pin_memory() for v in got)
        state["plan"] = swc.HostPlan(_ints(case["shape"]), case["dtype"], _ints(case["window"]), 1,
                                     case["border"], band_rows=case["band"], depth=case["depth"])
        state["out"] = torch.empty(_ints(case["shape"]), dtype=torch.float32, pin_memory=True)
    else:
        state["x"], state["y"] = got
    if "window" in case:
        state["window"] = _ints(case["window"])
    if "step" in case:
        state["step"] = _ints(case["step"])
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "batch":
        c = state["plan"].launch()
        return dict(c=list(c), flags=list(state["plan"].flags)) if case["flags"] else list(c)
    if case["kind"] == "filter":
        c, flags = swc.corr(state["x"], state["y"], state["window"], return_flags=True)
        return dict(c=c, flags=flags, mask=swc.cloud_mask(c, flags, case["tau"]),
                    keep=swc.filter_detections(c, state["idx"], flags, case["tau"]))
    if case["kind"] == "host":
        return state["plan"].run(state["x"], state["y"], state["out"])[0]
    got = swc.corr(state["x"], state["y"], state["window"], state["step"], case["border"],
                   return_flags=case["flags"])
    return dict(c=got[0], flags=got[1]) if case["flags"] else got


# ---- what a pass cannot do without ------------------------------------------

def _out_shape(shape, window, step, border):
    return [(n - k) // s + 1 if border == "valid" else -(-n // s)
            for n, k, s in zip(shape, window, step)]


def work(case):
    """Inputs read once, outputs written once; per element three products and
    a moving sum (two additions of five channels) per axis, per output the
    formula."""
    if case["kind"] == "batch":
        parts = [((h, w), 2, 1.0) for h, w, _ in _batch_shapes(case)]
    else:
        parts = [(_ints(case["shape"]), len(_ints(case["shape"])), 1.0)]
    item = ITEM[case.get("dtype", "u16")]
    nbytes = flops = 0.0
    for shape, nd, _ in parts:
        n = math.prod(shape)
        o = n
        if "step" in case:
            o = math.prod(_out_shape(shape, _ints(case["window"]), _ints(case["step"]),
                                     case["border"]))
        nbytes += 2.0 * item * n + 4.0 * o + (o if case.get("flags") else 0)
        flops += n * (3.0 + 10.0 * nd) + 13.0 * o
        if case["kind"] == "filter":
            nbytes += 7.0 * o + 14.0 * case["detections"]
    return dict(bytes=nbytes, flops=flops)


# ---- the same in 64 bits ----------------------------------------------------

def _ends(n, k, s, border):
    """First and last (clipped) cell of every window along one axis, and
    whether the window crosses the array's edge."""
    count = (n - k) // s + 1 if border == "valid" else -(-n // s)
    lo = torch.arange(count, device="cuda") * s - (0 if border == "valid" else k // 2)
    hi = lo + k - 1
    return lo.clamp(min=0), hi.clamp(max=n - 1), (lo < 0) | (hi >= n)


def _box(v, ends):
    for d, (lo, hi, _) in enumerate(ends):
        c = torch.cumsum(v, d)
        v = c.index_select(d, hi)
        first = c.index_select(d, (lo - 1).clamp(min=0))
        shape = [1] * v.dim()
        shape[d] = -1
        v = v - first * (lo > 0).view(shape).to(v.dtype)
    return v


def _map(x, y, window, step, border):
    """Section 1's formula on window sums: exact integers for integer input,
    centred float64 for float input.  Invalid windows give -2."""
    ends = [_ends(n, k, s, border) for n, k, s in zip(x.shape, window, step)]
    n = None
    bad = None
    for d, (lo, hi, crosses) in enumerate(ends):
        shape = [1] * x.dim()
        shape[d] = -1
        cells = (hi - lo + 1).view(shape)
        n = cells if n is None else n * cells
        crosses = crosses.view(shape)
        bad = crosses if bad is None else bad | crosses
    if border != "fill":
        bad = torch.zeros_like(bad)
    if x.dtype == torch.float32:
        gone = ~((x > MISSING) & (y > MISSING) & torch.isfinite(x) & torch.isfinite(y))
        a, b = x.double(), y.double()
        a, b = (torch.where(gone, 0.0, v - v[~gone].mean()) for v in (a, b))
        bad = bad | (_box(gone.to(torch.int32), ends) > 0) | (n == 1)
    else:
        a, b = x.to(torch.int64), y.to(torch.int64)
    sa, sb = _box(a, ends), _box(b, ends)
    va = n * _box(a * a, ends) - sa * sa
    vb = n * _box(b * b, ends) - sb * sb
    cov = n * _box(a * b, ends) - sa * sb
    if x.dtype != torch.float32:
        bad = bad | (va == 0) | (vb == 0)
    c = cov.double() / (va.double() * vb.double()).sqrt()
    return torch.where(bad, INVALID, c.clamp(-1.0, 1.0))


def exact(case, seed):
    got = _inputs(case, seed)
    if case["kind"] == "batch":
        c = [_map(x, y, (k, k), (1, 1), "clip") for (x, y), (_, _, k) in zip(got, _batch_shapes(case))]
        return dict(c=c, flags=[None] * len(c)) if case["flags"] else c
    window = _ints(case["window"])
    step = _ints(case["step"]) if "step" in case else (1,) * len(window)
    c = _map(got[0], got[1], window, step, case.get("border", "fill"))
    if case["kind"] == "filter":
        return dict(c=c, flags=None, mask=None, keep=None)
    if case["kind"] == "host":
        return c
    return dict(c=c, flags=None) if case["flags"] else c
