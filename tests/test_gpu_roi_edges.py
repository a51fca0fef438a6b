"""ROI detection at the edges of its 16-byte units: widths below, at and above
a unit of every format, odd pitches, buffers that start at any pixel, data in
the columns past the image's width (which must not count), single pixels in
corners, and workspaces that only fit the coarse bands."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_08755_amd as cmp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
FMT = {"depth": cmp.RGBA8, "rgba8": cmp.RGBA8, "f32": cmp.RGBA32F, "f16": cmp.RGBA16F}


def _image(rng, fmt, w, h, pitch, shift):
    """An image at pixel `shift` of its buffer; everything around it is data."""
    where = rng.random((h, w)) < rng.choice([0.0, 2.0 / (w * h), 0.01, 0.3])
    for y, x in ((0, 0), (0, w - 1), (h - 1, 0), (h - 1, w - 1)):
        if rng.random() < 0.15:
            where[y, x] = True
    mask = np.ones(h * pitch + shift + 4, bool)
    view = mask[shift:shift + h * pitch].reshape(h, pitch)
    view[:, :w] = where
    if fmt in ("depth", "rgba8"):
        empty = 0xFFFFFFFF if fmt == "depth" else 0
        a = np.where(mask, 5, empty).astype(np.uint32)
        t = torch.from_numpy(a.view(np.int32)).to(DEV)[shift:shift + h * pitch].view(h, pitch)
        full = a[shift:shift + h * pitch].reshape(h, pitch)
        ref = (oracle.roi_detect_depth if fmt == "depth" else oracle.roi_detect_rgba8)(full, w, h)
        return cmp.Image(t, t if fmt == "depth" else None, (0, 0, w, h)), tuple(ref)
    a = np.zeros((mask.size, 4), np.float16 if fmt == "f16" else np.float32)
    a[:, 1] = -0.0
    a[mask, rng.integers(0, 4)] = 0.5
    t = torch.from_numpy(a).to(DEV)[shift:shift + h * pitch].view(h, pitch, 4)
    ref = oracle.roi_detect_rgbaf(a[shift:shift + h * pitch].reshape(h, pitch, 4), w, h)
    return cmp.Image(t, None, (0, 0, w, h)), tuple(ref)


@pytest.mark.parametrize("fmt", list(FMT))
@pytest.mark.parametrize("widths", [(1, 2, 3, 4, 5, 6, 7, 8, 9), (15, 16, 17, 255, 257, 1023, 1279),
                                    (4099,)])
def test_roi_unit_edges(fmt, widths):
    rng = np.random.default_rng(len(widths) * 10 + list(FMT).index(fmt))
    imgs, refs = [], []
    for k, w in enumerate(widths):
        for h in (1, 7, 61):
            img, ref = _image(rng, fmt, w, h, w + int(rng.integers(0, 4)), (k + h) % 4)
            imgs.append(img)
            refs.append(ref)
    print(f"[gpu case] roi unit edges {fmt} {widths}", flush=True)
    roi = cmp.roi_detect(imgs, fmt=FMT[fmt])
    # bands of 128 KiB: one slot per image here
    ws = torch.zeros(8192 + 16 * len(imgs), dtype=torch.uint8, device=DEV)
    coarse = None
    if max(im.roi[2] * im.roi[3] for im in imgs) * 16 <= 128 * 1024:
        coarse = cmp.roi_detect(imgs, fmt=FMT[fmt], ws=ws)
    torch.cuda.synchronize()
    assert [tuple(r) for r in roi.cpu().tolist()] == refs
    assert coarse is None or torch.equal(coarse, roi)


def test_roi_bands_of_a_large_launch():
    """More than 1000 bands of 128 KiB, so that larger ones are taken; and the
    same images with the least workspace that their 128 KiB bands need."""
    rng = np.random.default_rng(3)
    w, h, n = 3001, 2003, 8
    d = torch.full((n, h, w), -1, dtype=torch.int32, device=DEV)
    refs = []
    for i in range(n):
        (x0, x1), (y0, y1) = sorted(rng.integers(0, w, 2)), sorted(rng.integers(0, h, 2))
        d[i, y0, x1] = d[i, y1, x0] = 1
        refs.append((int(x0), int(y0), int(x1 - x0 + 1), int(y1 - y0 + 1)))
    imgs = [cmp.Image(d[i], d[i], (0, 0, w, h)) for i in range(n)]
    slots = n * -(-h // -(-128 * 1024 // (4 * w)))
    ws = torch.zeros(8192 + 16 * slots, dtype=torch.uint8, device=DEV)
    print("[gpu case] roi large launch", flush=True)
    for _ in range(2):
        for work in (None, ws):
            roi = cmp.roi_detect(imgs, ws=work)
            torch.cuda.synchronize()
            assert [tuple(r) for r in roi.cpu().tolist()] == refs
