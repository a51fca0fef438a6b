"""ROI detection of images narrower than a 16-byte unit over more rows than a
workgroup has in flight."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_08755_amd as cmp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("fmt,width", [("depth", 1), ("depth", 2), ("depth", 3), ("rgba8", 3),
                                       ("f16", 1)])
def test_roi_narrow_and_tall(fmt, width):
    rng = np.random.default_rng(width)
    imgs, refs = [], []
    for h in (1, 255, 257, 2047, 2048, 2049, 9001, 40000):
        for hits in (0, 1, 3):
            where = np.zeros((h, width), bool)
            for _ in range(hits):
                where[rng.integers(0, h), rng.integers(0, width)] = True
            full = np.ones((h, width + 2), bool)   # the columns past the width hold data
            full[:, :width] = where
            if fmt == "f16":
                a = np.zeros((*full.shape, 4), np.float16)
                a[full, 2] = 0.5
                refs.append(tuple(oracle.roi_detect_rgbaf(a, width, h)))
                t = torch.from_numpy(a).to(DEV)
            else:
                a = np.where(full, 5, 0xFFFFFFFF if fmt == "depth" else 0).astype(np.uint32)
                ref = oracle.roi_detect_depth if fmt == "depth" else oracle.roi_detect_rgba8
                refs.append(tuple(ref(a, width, h)))
                t = torch.from_numpy(a.view(np.int32)).to(DEV)
            imgs.append(cmp.Image(t, t if fmt == "depth" else None, (0, 0, width, h)))
    print(f"[gpu case] roi narrow {fmt} {width}", flush=True)
    roi = cmp.roi_detect(imgs, fmt=cmp.RGBA16F if fmt == "f16" else cmp.RGBA8)
    torch.cuda.synchronize()
    assert [tuple(r) for r in roi.cpu().tolist()] == refs
