"""Depth compositing at the edges of its passes: contributor counts around the
64 that a wave tests at a time and around what one launch takes (111 with one
region, 76 with 64; fewer where a pitch exceeds 32 bits), steps and tiles cut
by the viewport, tile counts around a run of the tile order, and placements at
the ends of the 32-bit range."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_08755_amd as cmp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _contributor(rng, x, y, w, h, pad):
    c = rng.integers(0, 1 << 32, size=(h, w + pad), dtype=np.uint32)
    d = rng.integers(0, 6, size=(h, w + pad)).astype(np.uint32)   # many ties
    d[rng.random((h, w + pad)) < 0.2] = 0xFFFFFFFF                # clear depth
    t = [torch.from_numpy(a.view(np.int32)).to(DEV) for a in (c, d)]
    return cmp.Image(t[0], t[1], (x, y, w, h)), c, d


def _check(items, vp, sched, note, images=None, **kw):
    print(f"[gpu case] depth passes {note} n={len(items)} {vp} {sched}", flush=True)
    oc, od = cmp.composite_depth(images or [i[0] for i in items], vp, schedule=sched, **kw)
    rc, rd = oracle.composite_depth([i[1] for i in items], [i[2] for i in items],
                                    [i[0].roi for i in items], vp)
    assert np.array_equal(oc.cpu().numpy().view(np.uint32), rc)
    assert np.array_equal(od.cpu().numpy().view(np.uint32), rd)


@pytest.mark.parametrize("n,W,H,sched", [
    (1, 1, 1, ("seq", 1)), (5, 65, 17, ("seq", 1)), (63, 130, 33, ("direct_send", 3)),
    (64, 64, 16, ("seq", 1)), (65, 63, 15, ("seq", 1)), (76, 200, 130, ("binary_swap", 64)),
    (77, 200, 130, ("binary_swap", 64)), (111, 129, 40, ("seq", 1)), (112, 129, 40, ("seq", 1)),
    (128, 70, 50, ("direct_send", 64)), (230, 90, 30, ("seq", 1)), (9, 700, 200, ("seq", 1)),
    (9, 1030, 500, ("direct_send", 5))])
def test_depth_passes(n, W, H, sched):
    rng = np.random.default_rng(10 * n + W)
    items = []
    for _ in range(n):
        w, h = int(rng.integers(1, W + 2)), int(rng.integers(1, H + 2))
        x, y = int(rng.integers(-w, W + 1)), int(rng.integers(-h, H + 1))
        items.append(_contributor(rng, x, y, w, h, int(rng.integers(0, 3))))
    _check(items, (0, 0, W, H), sched, "counts")
    _check(items, (-3, 2, W, H), sched, "shifted", tile=(24, 7))


def test_depth_far_and_wide():
    """Contributors at the ends of the 32-bit range do not reach the viewport;
    single rows whose pitch needs more than 32 bits do."""
    rng = np.random.default_rng(3)
    items = [_contributor(rng, -2, 1, 90, 6, 1), _contributor(rng, 10, 0, 40, 9, 0)]
    for x, y in [(2**31 - 3, 0), (-2**31, 0), (0, 2**31 - 2), (0, -2**31), (2**31 - 3, 2**31 - 2)]:
        items.append(_contributor(rng, x, y, 2, 1, 0))
    for k in range(101):   # more than one pass of contributors with wide pitches
        items.append(_contributor(rng, int(rng.integers(0, 60)), k % 8, 30, 1, 0))
    images = [i[0] for i in items]
    for k in range(7, len(images), 3):
        im = images[k]
        wide = [torch.as_strided(t, (1, 30), (2**32 + 64, 1)) for t in (im.color, im.depth)]
        images[k] = cmp.Image(wide[0], wide[1], im.roi)
    assert images[7].color.stride(0) > 2**32
    for sched in (("seq", 1), ("direct_send", 6)):
        _check(items, (0, 0, 100, 8), sched, "far and wide", images=images)


def test_depth_without_depth_output():
    """48 contributors without a depth output are one pass whatever the
    regions; 49 are refused."""
    rng = np.random.default_rng(4)
    items = [_contributor(rng, int(rng.integers(-5, 60)), int(rng.integers(-5, 30)), 30, 20, 1)
             for _ in range(49)]
    images = [i[0] for i in items]
    print("[gpu case] depth without depth output", flush=True)
    for sched in (("seq", 1), ("binary_swap", 64)):
        oc, od = cmp.composite_depth(images[:48], (0, 0, 80, 45), schedule=sched, want_depth=False)
        assert od is None
        rc, _ = oracle.composite_depth([i[1] for i in items[:48]], [i[2] for i in items[:48]],
                                       [i[0].roi for i in items[:48]], (0, 0, 80, 45))
        assert np.array_equal(oc.cpu().numpy().view(np.uint32), rc)
        with pytest.raises(cmp.CmpError):
            cmp.composite_depth(images, (0, 0, 80, 45), schedule=sched, want_depth=False)
