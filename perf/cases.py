"""The workloads this library is timed on, through its public entry points.

A case is a dict of plain values. ``listed()`` names the workloads; ``draw(rng)``
gives another one of the same ranges; ``prepare`` makes what a program holds
before the call, ``run`` makes one call, ``work`` counts what a call cannot do
without and ``exact`` computes the same outputs in 64 bits with plain torch.

Kinds of case:
  image   forward or inverse of one image, ``dwt.forward`` / ``dwt.inverse``
  level   one forward or inverse level into (from) separate bands
  batch   a planned batch of uneven images, levels 1 and 2 fused
  serve   a burst of mixed requests through the serving loop
"""
from __future__ import annotations

import math
import random

import torch

import paper_1705_08266_amd as dwt
from paper_1705_08266_amd.batch import BatchPlan
from paper_1705_08266_amd.serving import Request, Server

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def _image(name, w, h, levels, dtype, wavelet, inverse=False, reuse=False, pad=0,
           scheme="nonseparable"):
    c = dict(kind="image", width=w, height=h, levels=levels, dtype=dtype, wavelet=wavelet,
             inverse=inverse, reuse=reuse, pad=pad, scheme=scheme)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a thumbnail or a tile of a larger picture: the call itself is the cost
        _image("fwd_64_f32", 64, 64, 3, "f32", "cdf97"),
        # decoding one mid-size picture kept in half precision, the 5/3 wavelet
        _image("inv_512_f16_53", 512, 512, 4, "f16", "cdf53", inverse=True),
        # a screen-size picture whose rows are not a multiple of a vector
        _image("fwd_1366x768_f32_L1", 1366, 768, 1, "f32", "cdf97"),
        # a video frame: 1080 rows leave odd level heights (540, 270, 135)
        _image("inv_1080p_bf16", 1920, 1080, 3, "bf16", "cdf97", inverse=True),
        # the benchmark's image in each direction, buffers allocated once
        _image("fwd_4096_f32", 4096, 4096, 5, "f32", "cdf97", reuse=True),
        _image("inv_4096_f32", 4096, 4096, 5, "f32", "cdf97", inverse=True, reuse=True),
        # one level into separate bands, the building block of a program's own pyramid
        dict(name="level_4096_f32_53", kind="level", width=4096, height=4096, dtype="f32",
             wavelet="cdf53", inverse=False, scheme="nonseparable"),
        # an 8K frame in half precision
        _image("fwd_8k_f16", 7680, 4320, 5, "f16", "cdf97", reuse=True),
        # the largest images: one forward in FP32, one reconstruction in half precision
        _image("fwd_16384_f32", 16384, 16384, 5, "f32", "cdf97", reuse=True),
        _image("inv_16384_f16", 16384, 16384, 5, "f16", "cdf97", inverse=True, reuse=True),
        # many uneven images planned once (sides log-uniform in 64..4096)
        dict(name="batch_32_f32", kind="batch", images=32, lo=64, hi=4096, levels=3, dtype="f32",
             wavelet="cdf97", inverse=False, scheme="nonseparable", shapes=1),
        # a burst of requests at the server (square sides log-uniform in 256..8192)
        dict(name="serve_24_f16", kind="serve", requests=24, lo=256, hi=8192, dtype="f16",
             wavelet="cdf97", scheme="nonseparable", shapes=2),
    ]


def draw(rng):
    kind = rng.choices(["image", "level", "batch", "serve"], [14, 3, 2, 1])[0]
    dtype = rng.choice(["f32", "f32", "f16", "bf16"])
    wavelet = rng.choice(["cdf97", "cdf97", "cdf53"])
    scheme = rng.choice(["nonseparable"] * 5 + ["separable"])
    inverse = rng.random() < 0.5
    if kind == "batch":
        return dict(kind="batch", images=rng.randint(4, 32), lo=64, hi=rng.choice([512, 2048, 4096]),
                    levels=rng.randint(1, 4), dtype=dtype, wavelet=wavelet, inverse=inverse,
                    scheme=scheme, shapes=rng.randint(3, 1 << 20))
    if kind == "serve":
        return dict(kind="serve", requests=rng.randint(4, 24), lo=256, hi=rng.choice([1024, 4096]),
                    dtype=dtype, wavelet=wavelet, scheme=scheme, shapes=rng.randint(3, 1 << 20))
    levels = 1 if kind == "level" else rng.randint(1, 5)

    def side():
        s = math.exp(rng.uniform(math.log(16.0), math.log(16384.0)))
        return max(1, round(s / (1 << levels))) << levels

    # an aspect ratio of at most 8, as pictures have
    w = side()
    h = max(1, round(w * math.exp(rng.uniform(-math.log(8.0), math.log(8.0))) / (1 << levels)))
    h = min(h << levels, 16384)
    if kind == "level":
        return dict(kind="level", width=w, height=h, dtype=dtype, wavelet=wavelet,
                    inverse=inverse, scheme=scheme)
    pad = rng.choice([0, 0, 0, 0, 2, 7, 32])   # a crop of a wider picture
    return _image(None, w, h, levels, dtype, wavelet, inverse, rng.random() < 0.5, pad, scheme)


# ---- inputs ---------------------------------------------------------------------

def _picture(h, w, g):
    """Smooth waves with texture and noise in 0..255, as 8-bit photographs have."""
    dev = "cuda"
    p = torch.rand(4, 4, generator=g, device=dev)
    y = torch.arange(h, device=dev, dtype=torch.float32)[:, None]
    x = torch.arange(w, device=dev, dtype=torch.float32)[None, :]
    im = torch.randn(h, w, generator=g, device=dev).mul_(4).add_(128)
    for k in range(4):
        f = 2 * math.pi / (8.0 * 64.0 ** p[k, 0])
        a = math.pi * p[k, 1]
        # sin(u + v) from one row and one column of values each
        u, v = f * torch.cos(a) * x + 6.28 * p[k, 2], f * torch.sin(a) * y
        im.addmm_(torch.cat([torch.cos(v), torch.sin(v)], 1),
                  torch.cat([torch.sin(u), torch.cos(u)], 0), alpha=24.0)
    return im.clamp_(0, 255).round_()


def _strided(t, pad):
    """t, as a crop of a buffer whose rows are `pad` elements longer."""
    if not pad:
        return t
    wide = torch.zeros(t.shape[0], t.shape[1] + pad, dtype=t.dtype, device=t.device)
    wide[:, :t.shape[1]] = t
    return wide[:, :t.shape[1]]


def _generator(seed, k=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1009 + k)
    return g


def _input(h, w, levels, dtype, wavelet, inverse, g):
    im = _picture(h, w, g)
    if inverse:   # the pyramid of a picture, in the storage type
        im = _forward64(im.double(), wavelet, levels)
    return im.to(DTYPES[dtype])


def _log_uniform(r, lo, hi, multiple):
    s = math.exp(r.uniform(math.log(lo), math.log(hi)))
    return max(multiple, int(round(s / multiple)) * multiple)


def _batch_sizes(c):
    r = random.Random(c["shapes"])
    return [(_log_uniform(r, c["lo"], c["hi"], 32), _log_uniform(r, c["lo"], c["hi"], 32))
            for _ in range(c["images"])]


def _requests(c):
    r = random.Random(c["shapes"])
    return [Request(i, 0.0, s, s, r.randint(1, 6), r.random() < 0.5)
            for i, s in enumerate(_log_uniform(r, c["lo"], c["hi"], 64)
                                  for _ in range(c["requests"]))]


def prepare(c, seed):
    kind, t = c["kind"], DTYPES[c["dtype"]]
    if kind == "image":
        h, w = c["height"], c["width"]
        x = _strided(_input(h, w, c["levels"], c["dtype"], c["wavelet"], c["inverse"],
                            _generator(seed)), c["pad"])
        kept = {}
        if c["reuse"]:
            kept = dict(out=torch.empty(h, w, dtype=t, device="cuda"),
                        workspace=dwt.make_workspace(w, h, c["levels"]))
        return dict(case=c, x=x, kept=kept)
    if kind == "level":
        h, w = c["height"], c["width"]
        x = _input(h, w, 1, c["dtype"], c["wavelet"], c["inverse"], _generator(seed))
        if c["inverse"]:
            bands = [b.contiguous() for b in _quadrants(x)]
            return dict(case=c, x=bands, out=torch.empty(h, w, dtype=t, device="cuda"))
        return dict(case=c, x=x, out=[torch.empty(h // 2, w // 2, dtype=t, device="cuda")
                                      for _ in range(4)])
    if kind == "batch":
        xs = [_input(h, w, c["levels"], c["dtype"], c["wavelet"], c["inverse"],
                     _generator(seed, k)) for k, (h, w) in enumerate(_batch_sizes(c))]
        make = BatchPlan.inverse_of if c["inverse"] else BatchPlan.forward
        return dict(case=c, plan=make(xs, levels=c["levels"], wavelet=c["wavelet"],
                                      scheme=c["scheme"], fuse_head=True))
    reqs = _requests(c)
    xs = {q.rid: _input(q.height, q.width, q.levels, c["dtype"], c["wavelet"], q.inverse,
                        _generator(seed, q.rid)) for q in reqs}
    return dict(case=c, requests=reqs, inputs=xs,
                server=Server(wavelet=c["wavelet"], scheme=c["scheme"], dtype=c["dtype"]))


def run(s):
    c = s["case"]
    if c["kind"] == "image":
        f = dwt.inverse if c["inverse"] else dwt.forward
        return f(s["x"], c["wavelet"], levels=c["levels"], scheme=c["scheme"], **s["kept"])
    if c["kind"] == "level":
        if c["inverse"]:
            dwt.inverse_level(*s["x"], s["out"], c["wavelet"], c["scheme"])
        else:
            dwt.forward_level(s["x"], *s["out"], c["wavelet"], c["scheme"])
        return s["out"]
    if c["kind"] == "batch":
        s["plan"].run()
        return s["plan"].outputs
    results = s["server"].run(s["requests"], s["inputs"], keep_outputs=True, realtime=False)
    return [r.output for r in sorted(results, key=lambda r: r.rid)]


def work(c):
    """Bytes: each input read once and each output written once. Flops: the
    non-separable lifting's multiply-accumulates per 2x2 quad, every level."""
    per_quad = {"cdf97": 36, "cdf53": 18}[c["wavelet"]] * 2

    def one(w, h, levels):
        px = w * h
        return (2 * px * BYTES[c["dtype"]],
                per_quad * sum(px / 4 / 4 ** j for j in range(levels)))

    if c["kind"] in ("image", "level"):
        parts = [one(c["width"], c["height"], c.get("levels", 1))]
    elif c["kind"] == "batch":
        parts = [one(w, h, c["levels"]) for h, w in _batch_sizes(c)]
    else:
        parts = [one(q.width, q.height, q.levels) for q in _requests(c)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ---- 64-bit reference --------------------------------------------------------------
# Separable lifting over whole-sample symmetric extension, unit gain (low
# phase x 1/K, high phase x K/2; 5/3: 1 and 1/2), one axis at a time.
STEPS = {"cdf97": [(-1.586134342059924, -0.052980118572961),
                   (0.882911075530934, 0.443506852043971)],
         "cdf53": [(-0.5, 0.25)]}
GAIN = {"cdf97": (1 / 1.230174104914001, 1.230174104914001 / 2), "cdf53": (1.0, 0.5)}


def _shift(t, dim, forward):
    """Each line's next (previous) sample of the same phase, the edge one repeated: the
    symmetric extension seen from the other phase."""
    n = t.shape[dim]
    if forward:
        return torch.cat([t.narrow(dim, 1, n - 1), t.narrow(dim, n - 1, 1)], dim)
    return torch.cat([t.narrow(dim, 0, 1), t.narrow(dim, 0, n - 1)], dim)


def _split(x, wavelet, dim):
    e, o = (x[:, 0::2], x[:, 1::2]) if dim == 1 else (x[0::2], x[1::2])
    for p, u in STEPS[wavelet]:
        o = o + p * (e + _shift(e, dim, True))
        e = e + u * (o + _shift(o, dim, False))
    lo, hi = GAIN[wavelet]
    return e * lo, o * hi


def _merge(lo_band, hi_band, wavelet, dim):
    lo, hi = GAIN[wavelet]
    e, o = lo_band / lo, hi_band / hi
    for p, u in reversed(STEPS[wavelet]):
        e = e - u * (o + _shift(o, dim, False))
        o = o - p * (e + _shift(e, dim, True))
    return torch.stack([e, o], dim + 1).reshape(
        [n * 2 if d == dim else n for d, n in enumerate(e.shape)])


def _quadrants(x):
    h, w = x.shape[0] // 2, x.shape[1] // 2
    return x[:h, :w], x[:h, w:], x[h:, :w], x[h:, w:]


def _forward64(x, wavelet, levels):
    out = x.clone()
    for j in range(levels):
        v = out[:x.shape[0] >> j, :x.shape[1] >> j]
        lo, hi = _split(v, wavelet, 1)
        top, bottom = [torch.cat(b, 1) for b in zip(_split(lo, wavelet, 0),
                                                    _split(hi, wavelet, 0))]
        del lo, hi
        v.copy_(torch.cat([top, bottom], 0))
    return out


def _inverse64(x, wavelet, levels):
    out = x.clone()
    for j in reversed(range(levels)):
        v = out[:x.shape[0] >> j, :x.shape[1] >> j]
        ll, hl, lh, hh = _quadrants(v)
        v.copy_(_merge(_merge(ll, lh, wavelet, 0), _merge(hl, hh, wavelet, 0), wavelet, 1))
    return out


def exact(c, seed):
    s = prepare(c, seed)

    def of(x, levels, inverse):
        return (_inverse64 if inverse else _forward64)(x.double(), c["wavelet"], levels)

    if c["kind"] == "image":
        return of(s["x"], c["levels"], c["inverse"])
    if c["kind"] == "level":
        if c["inverse"]:
            ll, hl, lh, hh = s["x"]
            return of(torch.cat([torch.cat([ll, hl], 1), torch.cat([lh, hh], 1)], 0), 1, True)
        return list(_quadrants(of(s["x"], 1, False)))
    if c["kind"] == "batch":
        return [of(x, c["levels"], c["inverse"]) for x in s["plan"].srcs]
    return [of(s["inputs"][q.rid], q.levels, q.inverse) for q in s["requests"]]
