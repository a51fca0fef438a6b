"""Compression at the edges of its loads and stores, byte for byte against the
oracle: rectangles narrower and wider than a lane's 16 pixels, whose rows end
inside every quad position, in frames with a pitch; planes stored raw behind
run-coded planes of every size modulo 4; and more or fewer blocks than
workgroups, over images of very uneven size."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_08755_amd as cmp
import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _i32(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int32)).to(DEV)


def _frame(rng, W, H, P):
    """Runs in some bytes, noise in others, per frame."""
    def plane():
        kind = rng.integers(0, 3)
        if kind == 0:
            return rng.integers(0, 256, size=H * P, dtype=np.uint32)
        step = int(rng.integers(2, 40)) if kind == 1 else 700
        return np.repeat(rng.integers(0, 256, size=H * P // step + 1, dtype=np.uint32), step)[:H * P]
    words = [sum(plane() << (8 * k) for k in range(4)).astype(np.uint32).reshape(H, P)
             for _ in range(2)]
    return words


def _check(sizes, rois, seed, depth, swizzle):
    rng = np.random.default_rng(seed)
    imgs, host = [], []
    for W, H, P in sizes:
        c, d = _frame(rng, W, H, P)
        host.append((c[:, :W], d[:, :W] if depth else None))
        imgs.append(cmp.Image(_i32(c), _i32(d) if depth else None, (0, 0, W, H)))
    roi = torch.tensor(rois, dtype=torch.int32, device=DEV)
    print(f"[gpu case] rle edges seed={seed} n={len(sizes)} depth={depth} swizzle={swizzle}",
          flush=True)
    streams, n, st = cmp.rle_compress(imgs, roi_dev=roi, swizzle=swizzle)
    s64, n64, st64 = cmp.rle64_compress(imgs, roi_dev=roi)
    torch.cuda.synchronize()
    assert not st.any() and not st64.any()
    for i, (c, d) in enumerate(host):
        ref = oracle.rle_compress(c, d, tuple(rois[i]), swizzle=swizzle)
        assert int(n[i]) == ref.size and (streams[i][:ref.size].cpu().numpy() == ref).all(), i
        ref = oracle.rle64_compress(c, d, tuple(rois[i]))
        assert int(n64[i]) == ref.size and (s64[i][:ref.size].cpu().numpy() == ref).all(), i


@pytest.mark.parametrize("depth,swizzle", [(True, False), (False, False), (True, True)])
@pytest.mark.parametrize("w", [1, 3, 4, 15, 16, 17, 18, 19, 20, 31, 33, 62, 255, 257, 1001])
def test_rle_row_ends(w, depth, swizzle):
    h = -(-9000 // w)
    sizes = [(w + 5, h + 3, w + 8), (w + 2, h + 1, w + 2), (w, h, w + 1)]
    _check(sizes, [(3, 2, w, h), (1, 0, w, h), (0, 0, w, h)], w, depth, swizzle)


def test_rle_uneven_images():
    """One large image among small, one-pixel and empty ones, more blocks in
    all than workgroups; then as many blocks as images."""
    sizes = [(2600, 2000, 2600)] + [(64 + i, 70, 80 + i) for i in range(20)]
    rois = [(1, 3, 2597, 1990)] + [(i, 1, 64, 69) if i % 3 else (0, 0, 0, 0) for i in range(20)]
    rois[5] = (7, 7, 1, 1)
    _check(sizes, rois, 5, True, False)
    _check(sizes[1:], [(0, 0, 40, 3)] * 20, 6, True, False)
