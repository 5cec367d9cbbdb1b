"""The workloads whose speed is followed: single images, batches, 4D fields, the
smoothing pipeline and streaming, each through the public entry points.

``listed()`` gives the fixed cases, ``draw(rng)`` one more of the same ranges,
``prepare`` what a program holds before the call, ``run`` one pass, ``work`` the
bytes and operations the pass cannot do without, and ``exact`` the same outputs
from plain torch in 64 bits (every cell of the cubical complex counted).
"""
from __future__ import annotations

import itertools
import math

import numpy as np
import torch

from paper_2203_09087_amd import ecc, synth

DEVICE = "cuda"
ESIZE = {"u8": 1, "u16": 2, "f32": 4}
TAPS_SIGMA = 2.0


def listed():
    return [
        # a thumbnail or a tile of a 2D camera: one small call, launch latency
        dict(name="tile_u8", kind="single", shape="256x256", dtype="u8", texture="uniform", levels=256, bins=256,
             range="default", cons="vertex"),
        # a full-sky map projection (the paper's CMB images), the paper's filtration
        dict(name="map_u8_top", kind="single", shape="1500x3000", dtype="u8", texture="smooth", levels=256, bins=256,
             range="default", cons="top"),
        # a very large 2D scan, 12-bit levels in uint16, range found on the device
        dict(name="scan_u16", kind="single", shape="16384x16384", dtype="u16", texture="grf", levels=4096, bins=4096,
             range="auto", cons="vertex"),
        # a small reconstructed volume, 256 gray levels
        dict(name="volume_u8", kind="single", shape="256x256x256", dtype="u8", texture="smooth", levels=256,
             bins=256, range="default", cons="vertex"),
        # the large float field, known range
        dict(name="field_f32", kind="single", shape="512x512x512", dtype="f32", texture="grf", levels=0, bins=4096,
             range="explicit", cons="vertex"),
        # a float volume of odd sizes whose range is not known, the paper's filtration
        dict(name="field_f32_top", kind="single", shape="301x389x457", dtype="f32", texture="grf", levels=0,
             bins=1024, range="auto", cons="top"),
        # 16-bit data at a fine threshold grid (more bins than one LDS window)
        dict(name="fine_u16", kind="single", shape="190x310x263", dtype="u16", texture="grf", levels=65536,
             bins=16384, range="explicit", cons="vertex"),
        # the many-images workload: uneven 2D and 3D uint8 images, planned once
        dict(name="batch_u8", kind="plan", count=512, shapes_seed=5, dtype="u8", texture="smooth", levels=256,
             bins=256, range="default", cons="vertex"),
        # a serving batch: crops of uneven size that arrive together, one call
        dict(name="serve_u16", kind="batch", count=16, shapes_seed=6, dtype="u16", texture="grf", levels=4096,
             bins=4096, range="auto", cons="vertex"),
        # a time series of volumes as one 4D image
        dict(name="series_4d", kind="single", shape="8x256x256x256", dtype="f32", texture="grf", levels=0,
             bins=4096, range="auto", cons="vertex"),
        # smoothing + ECC, three steps of the paper's pipeline
        dict(name="pipeline", kind="pipeline", shape="1024x1024", steps=3, dtype="f32", texture="grf", levels=0,
             bins=1024, range="auto", cons="vertex"),
        # a volume that stays in pinned host memory and is streamed in slabs
        dict(name="stream_f32", kind="stream", shape="192x512x512", slab=64, dtype="f32", texture="grf", levels=0,
             bins=4096, range="explicit", cons="vertex"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _text(shape):
    return "x".join(str(n) for n in shape)


def draw(rng):
    kind = rng.choice(["2d", "2d", "3d", "3d", "3d", "4d", "plan", "batch", "pipeline", "stream"])
    cons = rng.choice(["vertex", "top"])
    dtype = rng.choice(["u8", "u16", "f32"])
    case = dict(kind="single", cons=cons, dtype=dtype)
    if dtype == "u8":
        case.update(texture=rng.choice(["smooth", "uniform"]), levels=256, bins=256, range="default")
    elif dtype == "u16":
        case.update(texture="grf", levels=rng.choice([4096, 65536]), bins=rng.choice([1024, 4096, 9000]),
                    range=rng.choice(["auto", "explicit"]))
    else:
        case.update(texture="grf", levels=0, bins=rng.choice([500, 1024, 4096]),
                    range=rng.choice(["auto", "explicit"]))
    if kind == "2d":
        case.update(shape=_text([_log_int(rng, 64, 8192) for _ in range(2)]))
    elif kind == "3d":
        case.update(shape=_text([_log_int(rng, 24, 500) for _ in range(3)]))
    elif kind == "4d":
        case.update(shape=_text([rng.randint(2, 8)] + [_log_int(rng, 24, 200) for _ in range(3)]))
    elif kind in ("plan", "batch"):
        case.update(kind=kind, count=_log_int(rng, 2, 128), shapes_seed=rng.randint(1, 10 ** 6))
        if case["bins"] > 4096:
            case["bins"] = 4096
    elif kind == "pipeline":
        case.update(kind="pipeline", shape=_text([_log_int(rng, 300, 2048) for _ in range(2)]),
                    steps=rng.randint(1, 4), dtype="f32", texture="grf", levels=0, bins=1024, range="auto")
    else:
        case.update(kind="stream", shape=_text([rng.randint(40, 160)] + [_log_int(rng, 100, 512) for _ in range(2)]),
                    slab=rng.choice([0, 16, 50]))
    return case


# ------------------------------------------------------------------ inputs

def _filtered(shape, gen, amplitude):
    """White noise filtered in Fourier space, on the next powers of two, cropped."""
    tile = [max(16, 1 << (n - 1).bit_length()) for n in shape]
    f = torch.fft.rfftn(torch.randn(tile, generator=gen, device=DEVICE))
    ks = [torch.fft.fftfreq(n, device=DEVICE) for n in tile[:-1]] + [torch.fft.rfftfreq(tile[-1], device=DEVICE)]
    k2 = torch.zeros(f.shape, device=DEVICE)
    for axis, k in enumerate(ks):
        k2 += (k * k).view([-1 if a == axis else 1 for a in range(len(tile))])
    f *= amplitude(k2)
    x = torch.fft.irfftn(f, s=tile)
    return x[tuple(slice(0, n) for n in shape)].contiguous()


def _noise(shape, texture, gen):
    if texture == "uniform":
        return torch.rand(shape, generator=gen, device=DEVICE)
    if texture == "smooth":     # white noise after a Gaussian of sigma 2
        return _filtered(shape, gen, lambda k2: torch.exp(k2 * (-2.0 * math.pi ** 2 * 4.0)))
    # a Gaussian random field with power spectrum k^-3, zero mean
    return _filtered(shape, gen, lambda k2: torch.where(k2 > 0, k2.clamp_min(1e-30) ** -0.75, torch.zeros_like(k2)))


def _levels(x, levels, dtype):
    """Min-max quantization to integer levels (uint16 data as its int16 bits)."""
    lo, hi = x.min(), x.max()
    q = ((x - lo) * (levels / (hi - lo).clamp_min(1e-30))).floor_().clamp_(0, levels - 1)
    if dtype == "u8":
        return q.to(torch.uint8)
    return q.to(torch.int32).to(torch.int16)


def _typed(x, case):
    return x if case["dtype"] == "f32" else _levels(x, case["levels"], case["dtype"])


def _shapes(case):
    if "shape" in case:
        return [tuple(int(n) for n in case["shape"].split("x"))]
    if case["kind"] == "plan":
        return synth.batch_shapes(count=case["count"], seed=case["shapes_seed"])
    reqs = synth.serving_requests(1000.0, case["count"], seed=case["shapes_seed"], side2d=(128, 2048), side3d=(32, 256))
    return [r["shape"] for r in reqs]


def _inputs(case, seed):
    """The case's images on the device: one drawn as such, or crops of two pools."""
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    shapes = _shapes(case)
    if "shape" in case:
        return [_typed(_noise(shapes[0], case["texture"], gen), case)]
    pools = {2: _noise((2048, 2048), case["texture"], gen), 3: _noise((256, 256, 256), case["texture"], gen)}
    offs = np.random.default_rng(seed)
    out = []
    for s in shapes:
        pool = pools[len(s)]
        at = [int(offs.integers(0, p - n + 1)) for p, n in zip(pool.shape, s)]
        out.append(_typed(pool[tuple(slice(a, a + n) for a, n in zip(at, s))].contiguous(), case))
    return out


def _range(case, image):
    """The range argument of the call: None, "auto", or (lo, hi)."""
    if case["range"] == "default":
        return None
    if case["range"] == "auto":
        return "auto"
    if case["dtype"] == "f32":
        return (float(image.min()), float(image.max()))
    return (0, case["levels"] - 1)


def _taps():
    w = np.exp(-0.5 * (np.arange(-6, 7) / TAPS_SIGMA) ** 2)
    return [float(v) for v in (w / w.sum()).astype(np.float32)]


# --------------------------------------------------------------- the passes

def prepare(case, seed):
    ctx = ecc.Context(0, case["cons"])
    ctx.reserve(32 << 20, 1 << 20)
    images = _inputs(case, seed)
    state = dict(case=case, ctx=ctx, images=images, ranges=[_range(case, x) for x in images])
    if case["kind"] == "plan":
        state["out"] = torch.empty((len(images), case["bins"]), dtype=torch.int64, device=DEVICE)
        state["plan"] = ctx.plan_batch(images, case["bins"], state["ranges"], outs=list(state["out"]))
    elif case["kind"] == "pipeline":
        state["taps"] = _taps()
    elif case["kind"] == "stream":
        host = torch.empty(images[0].shape, dtype=images[0].dtype, pin_memory=True)
        host.copy_(images[0])
        state["images"] = [host]
    return state


def run(state):
    case, ctx, images = state["case"], state["ctx"], state["images"]
    kind, bins = case["kind"], case["bins"]
    if kind == "plan":
        state["plan"].launch()
        return state["out"]
    if kind == "batch":
        out = torch.empty((len(images), bins), dtype=torch.int64, device=DEVICE)
        ctx.compute_batch(images, bins, state["ranges"], outs=list(out))
        return out
    if kind == "stream":
        return ctx.compute_streamed(images[0], bins, state["ranges"][0], slab_planes=case["slab"])
    if kind == "pipeline":
        x, curves = images[0], []
        for _ in range(case["steps"]):
            curves.append(ctx.compute(x, bins, "auto"))
            x = ctx.smooth13(x, state["taps"])
        return curves + [x]
    return ctx.compute(images[0], bins, state["ranges"][0])


def work(case):
    """Images read once, curves (and the smoothed image) written once; a cell of
    the complex is one comparison and one count."""
    byt = ops = 0
    for s in _shapes(case):
        n = math.prod(s)
        byt += n * ESIZE[case["dtype"]] + 8 * case["bins"]
        ops += n * 2 * 2 ** len(s)
        if case["kind"] == "pipeline":
            byt += n * 4 + 8 * case["bins"] * (case["steps"] - 1)
            ops += n * (52 * case["steps"] + 8 * (case["steps"] - 1))
    return {"bytes": byt, "flops": ops}


# ---------------------------------------------------- the same in 64 bits

def _bins(x, case, rng):
    nb = case["bins"]
    if case["dtype"] == "f32":
        v = x.double()
        lo, hi = (float(x.min()), float(x.max())) if rng == "auto" else rng
        return ((v - lo) * (nb / (hi - lo))).floor_().clamp_(0, nb - 1).int()
    v = x.int() & (0xFF if case["dtype"] == "u8" else 0xFFFF)
    lo, hi = (0, 255) if rng is None else ((int(v.min()), int(v.max())) if rng == "auto" else rng)
    return torch.div((v.clamp(lo, hi) - lo).long() * nb, hi - lo + 1, rounding_mode="floor").int()


def _curve(x, case, rng):
    """The ECC of one image: every cell counted at its value with its sign."""
    nb, d, top = case["bins"], x.dim(), case["cons"] == "top"
    b = _bins(x, case, rng)
    vcec = torch.zeros(nb, dtype=torch.int64, device=x.device)
    for pairs in itertools.product([False, True], repeat=d):
        c = b
        for axis, pair in enumerate(pairs):
            n = c.shape[axis]
            if not pair:
                continue
            if top:     # lattice points: the smaller neighbour, the only one at an end
                mid = torch.minimum(c.narrow(axis, 0, n - 1), c.narrow(axis, 1, n - 1))
                c = torch.cat([c.narrow(axis, 0, 1), mid, c.narrow(axis, n - 1, 1)], axis)
            else:       # edges: the larger end
                c = torch.maximum(c.narrow(axis, 0, n - 1), c.narrow(axis, 1, n - 1))
        dim = d - sum(pairs) if top else sum(pairs)
        if c.numel():
            vcec += (-1) ** dim * torch.bincount(c.reshape(-1), minlength=nb)
    return vcec.cumsum(0)


def _smooth64(x, taps):
    for axis in (1, 0):
        n = x.shape[axis]
        at = torch.arange(n, device=x.device)
        acc = torch.zeros_like(x)
        for k, w in enumerate(taps):
            acc += w * x.index_select(axis, (at + (k - 6)).clamp_(0, n - 1))
        x = acc
    return x


def exact(case, seed):
    images = _inputs(case, seed)
    ranges = [_range(case, x) for x in images]
    if case["kind"] == "pipeline":
        # the later curves bin images already rounded to float32: no 64-bit value
        x = images[0].double()
        for _ in range(case["steps"]):
            x = _smooth64(x, _taps())
        return [_curve(images[0], case, "auto")] + [None] * (case["steps"] - 1) + [x]
    curves = [_curve(x, case, r) for x, r in zip(images, ranges)]
    return torch.stack(curves) if case["kind"] in ("plan", "batch") else curves[0]
