"""Ordered compositing at the edges of its row segments and load batches: the
last segment of a row, layer counts around the batch sizes (2, 4, 8 FP32
layers; 4, 8, 16 FP16 layers), groups without layers, requested tiles that are
run as wider ones, and placements at the ends of the 32-bit range."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_08755_amd as cmp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _layers(rng, n, W, H, dtype):
    out = []
    for i in range(n):
        w, h = int(rng.integers(max(1, W // 2), W + 1)), int(rng.integers(max(1, H // 2), H + 1))
        x, y = int(rng.integers(-3, W - w + 4)), int(rng.integers(-2, H - h + 3))
        P = w + int(rng.integers(0, 3))
        a = rng.beta(2, 5, size=(h, P))
        L = np.concatenate([rng.random((h, P, 3)) * a[..., None], a[..., None]], -1)
        out.append(cmp.Image(torch.from_numpy(L.astype(dtype)).to(DEV), None, (x, y, w, h)))
    return out


@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("n,W,H", [(1, 1, 1), (2, 63, 3), (3, 64, 5), (4, 65, 4), (5, 127, 2),
                                   (8, 128, 9), (9, 129, 4), (15, 200, 3), (16, 64, 17),
                                   (17, 70, 5), (33, 191, 2), (64, 130, 3), (65, 66, 3)])
def test_over_segments(dtype, n, W, H):
    rng = np.random.default_rng(1000 * n + W)
    layers = _layers(rng, n, W, H, dtype)
    order = [int(v) for v in rng.permutation(n)]
    vp = (-1, 1, W, H)
    arrs, rois = [l.color.cpu().numpy() for l in layers], [l.roi for l in layers]
    ref = oracle.composite_over(arrs, rois, order, vp)
    print(f"[gpu case] over segments {dtype.__name__} n={n} {W}x{H}", flush=True)
    seq = cmp.composite_over(layers, order, vp)
    for tile in [(16, 16), (100, 3), (128, 1), (256, 4), (1, 7)]:
        assert torch.equal(cmp.composite_over(layers, order, vp, tile=tile), seq), tile
    got = seq.cpu().numpy().astype(np.float64)
    # n FP32 multiply-adds of non-negative terms: the library's stated bound
    assert (np.abs(got - ref) <= 2e-6 * np.abs(ref) + 1e-30).all()
    if n > 64:
        return
    for P in (1, 2, 8, 64):   # 64: groups without layers
        out = cmp.composite_over(layers, order, vp, schedule=("binary_swap", P))
        tree = oracle.composite_over(arrs, rois, order, vp, groups=P)
        got = out.cpu().numpy().astype(np.float64)
        assert (np.abs(got - tree) <= 2e-6 * np.abs(tree) + 1e-30).all(), P


def test_over_far_placements():
    """Layers placed at the ends of the 32-bit range do not reach the viewport."""
    rng = np.random.default_rng(7)
    near = _layers(rng, 3, 90, 6, np.float32)
    block = near[0].color[:1, :2].contiguous()
    far = [cmp.Image(block, None, (x, y, 2, 1))
           for x, y in [(-2**31, 0), (2**31 - 3, 0), (0, -2**31), (0, 2**31 - 2),
                        (-2**31, 2**31 - 2)]]
    vp = (-5, -3, 90, 6)
    print("[gpu case] over far placements", flush=True)
    ref = cmp.composite_over(near, [2, 0, 1], vp)
    out = cmp.composite_over(near + far, [4, 2, 3, 0, 5, 1, 6, 7], vp)
    assert torch.equal(out, ref)
