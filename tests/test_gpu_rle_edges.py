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
    # decoded into frames from buffers of the streams' own sizes; nothing
    # outside the rectangles is written
    exact = [s[:int(k)].clone() for s, k in zip(streams, n.tolist())]
    outs = [cmp.Image(torch.full((H, W), 7, dtype=torch.int32, device=DEV),
                      torch.full((H, W), 7, dtype=torch.int32, device=DEV) if depth else None,
                      (0, 0, W, H)) for W, H, _ in sizes]
    got, st = cmp.rle_decompress(exact, outs, at_roi=True)
    torch.cuda.synchronize()
    assert not st.any() and (got.cpu() == roi.cpu()).all()
    for i, (c, d) in enumerate(host):
        x, y, w, h = rois[i]
        for t, src in ((outs[i].color, c), (outs[i].depth, d)):
            if src is not None:
                want = np.full(src.shape, 7, np.uint32)
                want[y:y + h, x:x + w] = src[y:y + h, x:x + w]
                assert (synth.as_u32(t) == want).all(), i


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


def _set_token(stream, plane, index, length):
    """Overwrites the run length byte of a token of block 0."""
    s = stream.copy()
    nb, np_ = int(s[28:32].view(np.uint32)[0]), int(s[20])
    p0 = -(-(32 + 4 * nb * (1 + np_)) // 16) * 16
    size = s[32 + 4 * nb:32 + 4 * nb + 4 * np_].view(np.uint32)
    s[p0 + int(size[:plane].sum()) + 2 * index] = length - 1
    return s, int(size[plane]) // 2


def test_rle_decode_rejects_wrong_lengths():
    """A segment's token shorter or longer than the segment, in the first and
    in the last (shorter) segment, and a plane whose run lengths sum to the
    block's length plus 2^16."""
    H, W = 3, 700   # 2100 pixels: the last segment has 52
    color = np.zeros((H, W), np.uint32)
    runs = np.arange(H * W) * 272 // (H * W)          # 272 runs in byte 1
    cuts = np.concatenate([[0], np.flatnonzero(np.diff(runs)) + 1])
    color |= (runs.reshape(H, W).astype(np.uint32) & 0xFF) << 8
    ref = oracle.rle_compress(color, None, (0, 0, W, H))
    bad = []
    for index, length in ((0, 255), (3, 1), (8, 51), (8, 53), (8, 256)):
        s, ntok = _set_token(ref, 0, index, length)
        assert ntok == 9
        bad.append(s)
    # 4096 pixels: 272 whole-segment runs sum to 69632 = 4096 + 65536
    H2, W2 = 16, 256
    c2 = np.zeros((H2, W2), np.uint32)
    c2 |= ((np.arange(4096) // 16).reshape(H2, W2).astype(np.uint32) & 0xFF) << 8
    c2[0, 1:17] |= (np.arange(16, dtype=np.uint32) + 1) << 8
    s = oracle.rle_compress(c2, None, (0, 0, W2, H2))
    _, ntok = _set_token(s, 1, 0, 1)
    assert ntok == 272, ntok
    for i in range(ntok):
        s, _ = _set_token(s, 1, i, 256)
    print("[gpu case] rle wrong lengths", flush=True)
    streams = [torch.from_numpy(x.copy()).to(DEV) for x in [ref] + bad + [s]]
    outs = [cmp.Image(torch.zeros((H2, W), dtype=torch.int32, device=DEV), None, (0, 0, W, H2))
            for _ in streams]
    _, st = cmp.rle_decompress(streams, outs)
    torch.cuda.synchronize()
    assert st.cpu().tolist() == [0] + [cmp.CMP_ECORRUPT] * 6
    assert (synth.as_u32(outs[0].color)[:H] == color).all() and cuts.size == 272
