"""RL64 decompression writes four pixels per lane, 256 apart: rows shorter than
a quad, than 256 pixels and longer, odd sizes, a last pixel without a partner,
raw and token streams in one block, and frames with a wider pitch, of which
nothing beside the ROI may change."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_08755_amd as cmp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _plane(rng, w, h, mode):
    if mode == "raw":
        return rng.integers(0, 1 << 32, size=(h, w), dtype=np.uint32)
    if mode == "flat":
        return np.full((h, w), 0x01020304, np.uint32)
    v = np.repeat(rng.integers(0, 1 << 32, size=(w * h + 6) // 7 + 1, dtype=np.uint32),
                  rng.integers(1, 14, size=(w * h + 6) // 7 + 1))
    return np.resize(v, (h, w)).astype(np.uint32)


@pytest.mark.parametrize("modes", [("raw", "raw"), ("runs", "raw"), ("raw", "runs"),
                                   ("runs", "flat"), ("runs", None), ("raw", None)])
def test_rows(modes):
    rng = np.random.default_rng(17)
    sizes = [(1, 1), (1, 5000), (2, 4097), (3, 2731), (4, 1025), (5, 821), (63, 66), (64, 64),
             (253, 17), (255, 33), (256, 32), (257, 31), (1023, 9), (4095, 3), (4096, 2),
             (4097, 2), (9001, 1)]
    print(f"[gpu case] rl64 rows {modes}", flush=True)
    for pad in (0, 3):
        imgs, outs, refs = [], [], []
        for w, h in sizes:
            p = [_plane(rng, w, h, m) if m else None for m in modes]
            imgs.append(cmp.Image(*[None if a is None else torch.from_numpy(a.view(np.int32)).to(DEV)
                                    for a in p], (0, 0, w, h)))
            outs.append(cmp.Image(*[None if a is None else
                                    torch.full((h + 1, w + pad), 5, dtype=torch.int32, device=DEV)
                                    for a in p], (0, 0, w, h)))
            refs.append(p)
        streams, nbytes, status = cmp.rle64_compress(imgs)
        assert int(status.abs().sum()) == 0
        for s, n, p, (w, h) in zip(streams, nbytes.tolist(), refs, sizes):
            assert (s[:n].cpu().numpy() == oracle.rle64_compress(p[0], p[1], (0, 0, w, h))).all()
        _, st = cmp.rle64_decompress([s[:n].clone() for s, n in zip(streams, nbytes.tolist())], outs)
        assert (st == 0).all()
        for im, o, (w, h) in zip(imgs, outs, sizes):
            for a, b in ((im.color, o.color), (im.depth, o.depth)):
                if a is None:
                    continue
                assert torch.equal(b[:h, :w], a), (w, h)
                assert bool((b[h:] == 5).all()) and bool((b[:, w:] == 5).all()), (w, h)


def test_partner_of_an_odd_last_pixel():
    """A stream whose last symbol has a second pixel is malformed, token-coded
    or raw, and its block is not written."""
    rng = np.random.default_rng(5)
    for mode in ("raw", "runs"):
        w, h = 71, 3
        p = _plane(rng, w, h, mode)
        stream = oracle.rle64_compress(p, None, (0, 0, w, h)).copy()
        used = 32 + 8   # header, block offset and stream size
        payload = (used + 15) // 16 * 16
        size = int(stream[36:40].view(np.uint32)[0])
        for bad in (0, 1):
            s = stream.copy()
            if bad:
                s[payload + size - 1] ^= 0x40   # the upper word of the last value
            out = cmp.Image(torch.full((h, w), 5, dtype=torch.int32, device=DEV), None, (0, 0, w, h))
            print(f"[gpu case] rl64 partner {mode} {bad}", flush=True)
            _, st = cmp.rle64_decompress([torch.from_numpy(s).to(DEV)], [out])
            assert int(st[0]) == (cmp.CMP_ECORRUPT if bad else 0)
            if bad:
                assert bool((out.color == 5).all())
            else:
                assert (out.color.cpu().numpy().view(np.uint32) == p).all()
