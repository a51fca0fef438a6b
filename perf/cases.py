"""Performance cases of the compositing library: the calls that a sort-last
renderer makes, over the range of sizes it makes them at.

A case is a dict of plain values; ``prepare`` makes what the renderer holds
before the call (frames or layers in HBM, output buffers, marshalled call
arguments, the batch plan), ``run`` is one pass through the public entry
points, ``work`` the bytes and operations that pass cannot do without, and
``exact`` the float results in 64 bits. The kinds of case:

  depth   depth compositing of ROI-placed contributors
  frame   a whole sort-last frame: ROI detection, RLE compression,
          decompression into frames, depth compositing of their ROIs
  encode  per-component RLE compression of the detected ROIs
  decode  decompression of such streams into frames
  rl64    the two-pixel codec there and back
  over    ordered alpha compositing
  train   ordered compositing, a squared loss and its gradients
  batch   many uneven jobs in one persistent launch

Rendered data is synthetic: colour gradients and smooth depth ramps with a
little noise inside each contributor's rectangle on a clear frame, and volume
layers with alpha ~ Beta(2, 5) and premultiplied colour.
"""
import ctypes
import math
import random

import torch

import paper_1902_08755_amd as cmp

ENCODED = 2.6   # bytes per pixel of the per-component streams of these frames


def listed():
    return [
        # an interactive window with a handful of GPUs: latency counts
        dict(name="depth_4x640x480", kind="depth", n=4, w=640, h=480, area_lo=1.0, area_hi=1.0,
             schedule="seq", owners=1, marshalled=False),
        # a full-HD window rendered by a large cluster: many small ROIs, more
        # contributors than one launch takes
        dict(name="depth_100x1920x1080", kind="depth", n=100, w=1920, h=1080, area_lo=0.05,
             area_hi=0.2, schedule="direct_send", owners=16, marshalled=True),
        # the frame loop of 16 contributors at full HD
        dict(name="frame_16x1920x1080", kind="frame", n=16, w=1920, h=1080, area_lo=0.25,
             area_hi=0.35, owners=16),
        # the same loop in a window that the user has resized to odd sizes
        dict(name="frame_24x1279x719", kind="frame", n=24, w=1279, h=719, area_lo=0.05,
             area_hi=0.3, owners=8),
        # the sending side of a 4K wall
        dict(name="encode_8x3840x2160", kind="encode", n=8, w=3840, h=2160, area_lo=0.25,
             area_hi=0.35, depth=True, swizzle=False),
        # and its receiving side
        dict(name="decode_8x3840x2160", kind="decode", n=8, w=3840, h=2160, area_lo=0.25,
             area_hi=0.35, depth=True, swizzle=False),
        # the basic codec, both directions
        dict(name="rl64_8x1920x1080", kind="rl64", n=8, w=1920, h=1080, area_lo=0.25,
             area_hi=0.35),
        # full-screen volume slabs at 4K: the largest call
        dict(name="over_64x3840x2160_f32", kind="over", n=64, w=3840, h=2160, dtype="f32",
             frac_lo=1.0, frac_hi=1.0, schedule="seq", owners=1),
        # half-precision bricks of partial size, merged in binary-swap order
        dict(name="over_40x1921x1081_f16", kind="over", n=40, w=1921, h=1081, dtype="f16",
             frac_lo=0.25, frac_hi=1.0, schedule="binary_swap", owners=8),
        # a training step of a differentiable compositor
        dict(name="train_32x1024x1024_f32", kind="train", n=32, w=1024, h=1024, dtype="f32",
             frac_lo=1.0, frac_hi=1.0, outside=False),
        # many half-precision bricks, some of them reaching out of the view
        dict(name="train_80x961x541_f16", kind="train", n=80, w=961, h=541, dtype="f16",
             frac_lo=0.25, frac_hi=0.75, outside=True),
        # the tiles and thumbnails of a render service, depth and alpha mixed
        dict(name="batch_256", kind="batch", n=256, side_lo=64, side_hi=2048, c_lo=2, c_hi=32),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def size(lo, hi, n, most):
        """A window of lo..hi columns (odd ones too) with n * w * h <= most."""
        w = log_int(lo, hi)
        h = max(16, int(w * rng.uniform(0.45, 1.0)))
        f = min(1.0, math.sqrt(most / (n * w * h)))
        return max(16, int(w * f)), max(16, int(h * f))

    kind = rng.choice(["depth", "depth", "frame", "frame", "encode", "decode", "rl64", "over",
                       "over", "train", "batch"])
    if kind == "depth":
        n = log_int(2, 128)
        w, h = size(320, 3840, n, 2e8)
        lo = rng.choice([0.05, 0.1, 0.25])
        return dict(kind=kind, n=n, w=w, h=h, area_lo=lo, area_hi=2 * lo,
                    schedule=rng.choice(["seq", "direct_send", "binary_swap"]),
                    owners=rng.choice([1, 4, 16]), marshalled=rng.random() < 0.5)
    if kind == "frame":
        n = log_int(2, 48)
        w, h = size(320, 3840, n, 1e8)
        lo = rng.choice([0.05, 0.25])
        return dict(kind=kind, n=n, w=w, h=h, area_lo=lo, area_hi=lo + 0.1,
                    owners=rng.choice([1, 4, 16]))
    if kind in ("encode", "decode"):
        n = log_int(1, 16)
        w, h = size(320, 3840, n, 7e7)
        return dict(kind=kind, n=n, w=w, h=h, area_lo=0.25, area_hi=rng.choice([0.35, 1.0]),
                    depth=rng.random() < 0.7, swizzle=rng.random() < 0.3)
    if kind == "rl64":
        n = log_int(1, 16)
        w, h = size(320, 3840, n, 5e7)
        return dict(kind=kind, n=n, w=w, h=h, area_lo=0.25, area_hi=0.35)
    if kind == "over":
        n = log_int(2, 64)
        w, h = size(256, 3840, n, 2.5e8)
        full = rng.random() < 0.3
        return dict(kind=kind, n=n, w=w, h=h, dtype=rng.choice(["f32", "f16"]),
                    frac_lo=1.0 if full else 0.25, frac_hi=1.0,
                    schedule=rng.choice(["seq", "direct_send", "binary_swap"]),
                    owners=rng.choice([4, 8, 16]))
    if kind == "train":
        n = log_int(4, 128)
        w, h = size(128, 1100, min(n, 60), 3e7)
        return dict(kind=kind, n=min(n, 60) if rng.random() < 0.7 else n, w=w // (1 + n // 90),
                    h=h // (1 + n // 90), dtype=rng.choice(["f32", "f16"]),
                    frac_lo=0.25, frac_hi=rng.choice([0.75, 1.0]), outside=rng.random() < 0.5)
    return dict(kind=kind, n=log_int(8, 200), side_lo=64, side_hi=rng.choice([256, 512, 1024]),
                c_lo=2, c_hi=rng.choice([8, 32]))


# ------------------------------------------------------------------ inputs
class State:
    """What the caller keeps between passes."""


def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _gen(seed):
    return torch.Generator(device=_dev()).manual_seed(seed % (1 << 31))


def _rect(rng, w, h, lo, hi):
    """A rectangle of lo..hi of the viewport's area inside it."""
    a, s = rng.uniform(lo, hi), rng.uniform(0.8, 1.25)
    rw = min(w, max(1, round(w * math.sqrt(a) * s)))
    rh = min(h, max(1, round(h * math.sqrt(a) / s)))
    return rng.randint(0, w - rw), rng.randint(0, h - rh), rw, rh


def _layout(case):
    """Where the layers or jobs of a case lie: the case's own, so that its
    gradients and results have the same shapes whatever the seed."""
    return random.Random(repr(sorted((k, v) for k, v in case.items() if k != "name")))


def _i32(t):
    return torch.where(t >= 1 << 31, t - (1 << 32), t).to(torch.int32)


def _ramp(rng, gen, index, w, h):
    """Colour and depth of a rendered w x h block."""
    yy = torch.arange(h, device=_dev()).view(-1, 1)
    xx = torch.arange(w, device=_dev()).view(1, -1)
    d = rng.randint(1 << 30, 3 << 30) + rng.randint(-4096, 4096) * xx + rng.randint(-4096, 4096) * yy
    d = (d + torch.randint(-128, 128, (h, w), generator=gen, device=_dev())).clamp(0, (1 << 32) - 2)
    c = (255 * xx) // max(1, w - 1) + ((255 * yy) // max(1, h - 1) << 8)
    return _i32(c + (16 * index % 256 << 16) + (255 << 24)), _i32(d)


def _frames(rng, gen, n, w, h, lo, hi, depth=True):
    """n clear w x h frames, each with one rendered rectangle."""
    color = torch.zeros((n, h, w), dtype=torch.int32, device=_dev())
    deps = torch.full((n, h, w), -1, dtype=torch.int32, device=_dev()) if depth else None
    for i in range(n):
        x, y, rw, rh = _rect(rng, w, h, lo, hi)
        c, d = _ramp(rng, gen, i, rw, rh)
        color[i, y:y + rh, x:x + rw] = c
        if depth:
            deps[i, y:y + rh, x:x + rw] = d
    return [cmp.Image(color[i], deps[i] if depth else None, (0, 0, w, h)) for i in range(n)]


def _blank(n, w, h, depth=True):
    """n frames to decode into, in one block of memory each for colour and depth."""
    color = torch.zeros((n, h, w), dtype=torch.int32, device=_dev())
    deps = torch.zeros((n, h, w), dtype=torch.int32, device=_dev()) if depth else None
    return color, deps, [cmp.Image(color[i], deps[i] if depth else None, (0, 0, w, h))
                         for i in range(n)]


def _brick(gen, w, h, dtype):
    """A volume layer: alpha the second smallest of six uniforms, colour u * alpha."""
    u = torch.rand((h, w, 6), generator=gen, device=_dev())
    lo, hi = torch.minimum(u[..., 0], u[..., 1]), torch.maximum(u[..., 0], u[..., 1])
    for k in range(2, 6):
        hi = torch.minimum(hi, torch.maximum(lo, u[..., k]))
        lo = torch.minimum(lo, u[..., k])
    out = torch.empty((h, w, 4), device=_dev())
    torch.mul(torch.rand((h, w, 3), generator=gen, device=_dev()), hi.unsqueeze(-1), out=out[..., :3])
    out[..., 3] = hi
    return out.to(dtype)


def _bricks(rng, gen, c):
    dtype = torch.float16 if c["dtype"] == "f16" else torch.float32
    layers = []
    for _ in range(c["n"]):
        w = min(c["w"], max(1, round(c["w"] * rng.uniform(c["frac_lo"], c["frac_hi"]))))
        h = min(c["h"], max(1, round(c["h"] * rng.uniform(c["frac_lo"], c["frac_hi"]))))
        if c.get("outside"):
            x, y = rng.randint(-(w // 4), c["w"] - w + w // 4), rng.randint(-(h // 4), c["h"] - h + h // 4)
        else:
            x, y = rng.randint(0, c["w"] - w), rng.randint(0, c["h"] - h)
        layers.append(cmp.Image(_brick(gen, w, h, dtype), None, (x, y, w, h)))
    order = list(range(c["n"]))
    rng.shuffle(order)
    return layers, order


def _arena(sizes):
    """Stream buffers of the given sizes in one zeroed block, 256-byte aligned."""
    at, o = [], 0
    for b in sizes:
        at.append(o)
        o += (b + 255) // 256 * 256
    buf = torch.zeros(o, dtype=torch.uint8, device=_dev())
    return buf, [buf[a:a + b] for a, b in zip(at, sizes)]


def _ok(st):
    if st != cmp.CMP_OK:
        raise cmp.CmpError(st, "libcmp", cmp.lib().cmp_last_error().decode())


def _ptrs(ts):
    return (ctypes.c_void_p * len(ts))(*[t.data_ptr() for t in ts])


def _bytes(ts):
    return (ctypes.c_uint64 * len(ts))(*[t.numel() for t in ts])


def _c_images(imgs):
    return (cmp.CImage * len(imgs))(*[
        cmp.CImage(im.color.data_ptr(), im.depth.data_ptr() if im.depth is not None else None,
                   im.color.stride(0), cmp.Rect(*im.roi)) for im in imgs])


def prepare(case, seed):
    rng, gen, s, kind = random.Random(seed), _gen(seed), State(), case["kind"]
    s.case = case
    {"depth": _prepare_depth, "frame": _prepare_frame, "encode": _prepare_codec,
     "decode": _prepare_codec, "rl64": _prepare_codec, "over": _prepare_over,
     "train": _prepare_train, "batch": _prepare_batch}[kind](s, case, rng, gen)
    return s


def run(s):
    return {"depth": _run_depth, "frame": _run_frame, "encode": _run_encode,
            "decode": _run_decode, "rl64": _run_rl64, "over": _run_over, "train": _run_train,
            "batch": _run_batch}[s.case["kind"]](s)


# ------------------------------------------------------------------- depth
def _prepare_depth(s, c, rng, gen):
    s.images = []
    for i in range(c["n"]):
        roi = _rect(rng, c["w"], c["h"], c["area_lo"], c["area_hi"])
        s.images.append(cmp.Image(*_ramp(rng, gen, i, roi[2], roi[3]), roi))
    s.viewport = (0, 0, c["w"], c["h"])
    if c["marshalled"]:   # a render loop keeps its call arguments
        s.arr = _c_images(s.images)
        s.color = torch.zeros((c["h"], c["w"]), dtype=torch.int32, device=_dev())
        s.depth = torch.zeros_like(s.color)
        s.sched = cmp.Schedule(cmp._SCHED[c["schedule"]], c["owners"])


def _run_depth(s):
    c = s.case
    if not c["marshalled"]:
        return cmp.composite_depth(s.images, s.viewport, schedule=(c["schedule"], c["owners"]))
    _ok(cmp.lib().cmp_composite_depth(s.arr, c["n"], None, cmp.Rect(*s.viewport),
                                      s.color.data_ptr(), s.depth.data_ptr(), c["w"], s.sched,
                                      cmp.Tile(0, 0), torch.cuda.current_stream().cuda_stream))
    return s.color, s.depth


# ------------------------------------------------------------------- frame
def _prepare_frame(s, c, rng, gen):
    n, w, h, L = c["n"], c["w"], c["h"], cmp.lib()
    s.images = _frames(rng, gen, n, w, h, c["area_lo"], c["area_hi"])
    s.arr = _c_images(s.images)
    s.roi = torch.zeros((n, 4), dtype=torch.int32, device=_dev())
    s.roi_ws = torch.zeros(L.cmp_roi_workspace_size(s.arr, n), dtype=torch.uint8, device=_dev())
    s.streams, outs = _arena([cmp.rle_max_size(w, h, 8)] * n)
    s.out_ptrs, s.caps = _ptrs(outs), _bytes(outs)
    s.sizes = torch.zeros(n, dtype=torch.int64, device=_dev())
    s.c_status = torch.zeros(n, dtype=torch.int32, device=_dev())
    s.rle_ws = torch.zeros(L.cmp_rle_workspace_size(s.arr, n), dtype=torch.uint8, device=_dev())
    _, _, s.placed = _blank(n, w, h)
    s.placed_arr = _c_images(s.placed)
    s.roi_dec = torch.zeros((n, 4), dtype=torch.int32, device=_dev())
    s.d_status = torch.zeros(n, dtype=torch.int32, device=_dev())
    s.color = torch.zeros((h, w), dtype=torch.int32, device=_dev())
    s.depth = torch.zeros((h, w), dtype=torch.int32, device=_dev())


def _run_frame(s):
    c, L = s.case, cmp.lib()
    n, q = c["n"], torch.cuda.current_stream().cuda_stream
    _ok(L.cmp_roi_detect(s.arr, n, cmp.RGBA8, s.roi.data_ptr(), s.roi_ws.data_ptr(),
                         s.roi_ws.numel(), q))
    _ok(L.cmp_rle_compress(s.arr, n, cmp.RGBA8, 0, s.roi.data_ptr(), s.out_ptrs, s.caps,
                           s.sizes.data_ptr(), s.c_status.data_ptr(), s.rle_ws.data_ptr(),
                           s.rle_ws.numel(), q))
    _ok(L.cmp_rle_decompress_at_roi(s.out_ptrs, s.caps, n, s.placed_arr, s.roi_dec.data_ptr(),
                                    s.d_status.data_ptr(), q))
    _ok(L.cmp_composite_depth_crop(s.placed_arr, n, s.roi_dec.data_ptr(),
                                   cmp.Rect(0, 0, c["w"], c["h"]), s.color.data_ptr(),
                                   s.depth.data_ptr(), c["w"],
                                   cmp.Schedule(cmp.BINARY_SWAP, c["owners"]), cmp.Tile(0, 0), q))
    return s.color, s.depth, s.roi, s.sizes, s.c_status, s.d_status, s.roi_dec


# ------------------------------------------------------------------ codecs
def _prepare_codec(s, c, rng, gen):
    n, w, h, depth = c["n"], c["w"], c["h"], c.get("depth", True)
    s.images = _frames(rng, gen, n, w, h, c["area_lo"], c["area_hi"], depth)
    s.roi = cmp.roi_detect(s.images)
    if c["kind"] != "rl64":
        s.streams, outs = _arena([cmp.rle_max_size(w, h, 8 if depth else 4)] * n)
        s.rle = cmp.RleBatch(s.images, roi_dev=s.roi, outs=outs, swizzle=c["swizzle"])
    if c["kind"] != "encode":
        s.color, s.depth, s.frames = _blank(n, w, h, depth)
    if c["kind"] == "decode":
        s.rle.run()
        # what a receiver holds: buffers of the streams' own sizes
        sizes = s.rle.sizes.tolist()
        _, s.received = _arena(sizes)
        for to, o, b in zip(s.received, s.rle.outs, sizes):
            to.copy_(o[:b])
        s.rle = s.streams = s.images = None


def _run_encode(s):
    _, sizes, status = s.rle.run()
    return s.streams, sizes, status


def _run_decode(s):
    roi, status = cmp.rle_decompress(s.received, s.frames, at_roi=True)
    return [t for t in (s.color, s.depth, roi, status) if t is not None]


def _run_rl64(s):
    streams, sizes, status = cmp.rle64_compress(s.images, roi_dev=s.roi)
    roi, d_status = cmp.rle64_decompress(streams, s.frames)
    return s.color, s.depth, roi, sizes, status, d_status


# ----------------------------------------------------------- over and train
def _prepare_over(s, c, rng, gen):
    s.layers, s.order = _bricks(_layout(c), gen, c)
    s.viewport = (0, 0, c["w"], c["h"])
    s.out = torch.zeros((c["h"], c["w"], 4), device=_dev())


def _run_over(s):
    return cmp.composite_over(s.layers, s.order, s.viewport, out=s.out,
                              schedule=(s.case["schedule"], s.case["owners"]))


def _prepare_train(s, c, rng, gen):
    layers, s.order = _bricks(_layout(c), gen, c)
    s.viewport = (0, 0, c["w"], c["h"])
    s.rois = [l.roi for l in layers]
    s.rgba = [l.color.requires_grad_(True) for l in layers]
    s.target = torch.rand((c["h"], c["w"], 4), generator=gen, device=_dev())


def _run_train(s):
    out = cmp.OverComposite.apply(s.order, s.viewport, s.rois, *s.rgba)
    grads = torch.autograd.grad(((out - s.target) ** 2).sum(), s.rgba)
    # an optimiser takes the gradients as they are; the many are handed back together
    return [out.detach(), *(grads if len(grads) <= 60 else [torch.cat([g.reshape(-1) for g in grads])])]


# ------------------------------------------------------------------- batch
class _Plan:
    def __init__(self, jobs, n):
        self.h = ctypes.c_void_p()
        _ok(cmp.lib().cmp_batch_plan_create(jobs, n, None, ctypes.byref(self.h)))

    def __del__(self):
        if self.h:
            cmp.lib().cmp_batch_plan_destroy(self.h)


def _prepare_batch(s, c, rng, gen):
    s.jobs = []   # (kind, viewport, inputs, order)
    at = _layout(c)
    for j in range(c["n"]):
        w, h = (round(math.exp(at.uniform(math.log(c["side_lo"]), math.log(c["side_hi"]))))
                for _ in range(2))
        imgs = []
        for i in range(at.randint(c["c_lo"], c["c_hi"])):
            rw, rh = (max(1, round(v * at.uniform(0.25, 1.0))) for v in (w, h))
            roi = (at.randint(0, w - rw), at.randint(0, h - rh), rw, rh)
            imgs.append(cmp.Image(*_ramp(rng, gen, i, rw, rh), roi) if j % 2 == 0 else
                        cmp.Image(_brick(gen, rw, rh, torch.float32), None, roi))
        order = list(range(len(imgs)))
        rng.shuffle(order)
        s.jobs.append((j % 2, (w, h), imgs, order))
    # every job's output in one block of memory: a batch of depth results, one of colour
    d_px = sum(w * h for k, (w, h), _, _ in s.jobs if k == 0)
    o_px = sum(w * h for k, (w, h), _, _ in s.jobs if k == 1)
    s.color, s.depth = (torch.zeros(d_px, dtype=torch.int32, device=_dev()) for _ in range(2))
    s.rgba = torch.zeros((max(1, o_px), 4), device=_dev())
    arr, s.keep, d_at, o_at = (cmp.CJob * c["n"])(), [], 0, 0
    for j, (k, (w, h), imgs, order) in enumerate(s.jobs):
        ims = (cmp.CImage * len(imgs))(*[
            cmp.CImage(im.color.data_ptr(), im.depth.data_ptr() if k == 0 else None,
                       im.color.shape[1], cmp.Rect(*im.roi)) for im in imgs])
        o = (ctypes.c_int32 * len(order))(*order)
        s.keep += [ims, o]
        arr[j] = cmp.CJob(k, cmp.RGBA8 if k == 0 else cmp.RGBA32F, len(imgs), ims,
                          None if k == 0 else o, cmp.Rect(0, 0, w, h),
                          s.color[d_at:].data_ptr() if k == 0 else s.rgba[o_at:].data_ptr(),
                          s.depth[d_at:].data_ptr() if k == 0 else None, w)
        if k == 0:
            d_at += w * h
        else:
            o_at += w * h
    s.plan = _Plan(arr, c["n"])
    s.ws = torch.zeros(cmp.lib().cmp_batch_workspace_size(s.plan.h), dtype=torch.uint8, device=_dev())
    _ok(cmp.lib().cmp_batch_upload(s.plan.h, s.ws.data_ptr(), s.ws.numel(),
                                   torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()


def _run_batch(s):
    _ok(cmp.lib().cmp_batch_run(s.plan.h, s.ws.data_ptr(), torch.cuda.current_stream().cuda_stream))
    return s.color, s.depth, s.rgba


# -------------------------------------------------------------------- work
def work(c):
    kind, n = c["kind"], c["n"]
    if kind == "batch":
        # sides log-uniform, ROI sides uniform in [1/4, 1] of them
        mean = (c["side_hi"] - c["side_lo"]) / math.log(c["side_hi"] / c["side_lo"])
        px, cover = mean * mean, (c["c_lo"] + c["c_hi"]) / 2 * 0.625 ** 2
        jobs_d, jobs_o = (n + 1) // 2, n // 2
        return {"bytes": jobs_d * px * (4 * cover + 4 + 8) + jobs_o * px * (16 * cover + 16),
                "flops": jobs_o * px * cover * 9}
    px = c["w"] * c["h"]
    if kind in ("over", "train"):
        item = 8 if c["dtype"] == "f16" else 16
        cover = n * px * ((c["frac_lo"] + c["frac_hi"]) / 2) ** 2
        if kind == "over":
            return {"bytes": item * cover + 16 * px, "flops": 9 * cover}
        # the layers in, the gradients out, the image, the target
        return {"bytes": 2 * item * cover + 32 * px, "flops": 40 * cover}
    roi = n * px * (c["area_lo"] + c["area_hi"]) / 2
    if kind == "depth":
        return {"bytes": 4 * roi + 12 * px, "flops": roi}
    rec = 8 if c.get("depth", True) else 4
    if kind in ("encode", "decode"):
        return {"bytes": (rec + ENCODED * rec / 8) * roi, "flops": rec * roi}
    if kind == "rl64":
        return {"bytes": 2 * (8 + 7.5) * roi, "flops": 4 * roi}
    # frame: every depth read for its ROI, the ROIs encoded, decoded and composited
    return {"bytes": 4 * n * px + 2 * (8 + ENCODED) * roi + 4 * roi + 12 * px, "flops": 18 * roi}


# ------------------------------------------------------------------- exact
def _over64(layers, order, w, h):
    acc = torch.zeros((h, w, 4), dtype=torch.float64, device=_dev())
    for j in order:
        x, y, lw, lh = layers[j].roi
        x0, y0, x1, y1 = max(0, x), max(0, y), min(w, x + lw), min(h, y + lh)
        if x1 > x0 and y1 > y0:
            L = layers[j].color[y0 - y:y1 - y, x0 - x:x1 - x].double()
            a = acc[y0:y1, x0:x1]
            a.mul_(1 - L[..., 3:]).add_(L)
    return acc


def _grads64(layers, order, w, h, target):
    out = _over64(layers, order, w, h)
    G, T = 2 * (out - target.double()), torch.ones((h, w, 1), dtype=torch.float64, device=_dev())
    # S: what lies behind each layer, found by taking the layers off back to front
    S, behind = torch.zeros_like(out), {}
    for j in order:
        x, y, lw, lh = layers[j].roi
        x0, y0, x1, y1 = max(0, x), max(0, y), min(w, x + lw), min(h, y + lh)
        if x1 > x0 and y1 > y0:
            L = layers[j].color[y0 - y:y1 - y, x0 - x:x1 - x].double()
            s = S[y0:y1, x0:x1]
            behind[j] = (G[y0:y1, x0:x1] * s).sum(-1, keepdim=True)
            s.mul_(1 - L[..., 3:]).add_(L)
    grads = [None] * len(layers)
    for j in reversed(order):
        x, y, lw, lh = layers[j].roi
        g = torch.zeros((lh, lw, 4), dtype=torch.float64, device=_dev())
        x0, y0, x1, y1 = max(0, x), max(0, y), min(w, x + lw), min(h, y + lh)
        if x1 > x0 and y1 > y0:
            t = T[y0:y1, x0:x1]
            v = G[y0:y1, x0:x1] * t
            v[..., 3:] -= t * behind[j]
            g[y0 - y:y1 - y, x0 - x:x1 - x] = v
            t.mul_(1 - layers[j].color[y0 - y:y1 - y, x0 - x:x1 - x, 3:].double())
        grads[j] = g
    return [out, *(grads if len(grads) <= 60 else [torch.cat([g.reshape(-1) for g in grads])])]


@torch.no_grad()
def exact(case, seed):
    c, s = case, None
    if c["kind"] == "over":
        s = prepare(c, seed)
        return _over64(s.layers, s.order, c["w"], c["h"])
    if c["kind"] == "train":
        s = prepare(c, seed)
        layers = [cmp.Image(t.detach(), None, r) for t, r in zip(s.rgba, s.rois)]
        return _grads64(layers, s.order, c["w"], c["h"], s.target)
    if c["kind"] == "batch":
        s = prepare(c, seed)
        outs = [_over64(imgs, order, w, h).reshape(-1, 4)
                for k, (w, h), imgs, order in s.jobs if k == 1]
        return None, None, torch.cat(outs) if outs else torch.zeros((1, 4), dtype=torch.float64)
    return None   # whole numbers: they are compared as they are
