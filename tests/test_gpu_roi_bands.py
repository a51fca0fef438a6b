"""ROI detection of images narrower than a 16-byte unit over more rows than a
workgroup has in flight, and in a workspace that holds the slots of 128 KiB
bands but not those of the finer ones that small images are cut into."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_08755_amd as cmp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
TICKETS = 8192   # bytes of a workspace before its slots


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


def _slots(sizes, band):
    rows = [-(-band // (4 * w)) for w, _ in sizes]
    return sum(-(-h // r) for (_, h), r in zip(sizes, rows))


def test_roi_workspace_of_the_coarse_bands():
    rng = np.random.default_rng(1)
    sizes = [(575, 500), (600, 437), (511, 613), (575, 500)]   # 1.0 to 1.3 MB: bands of 32 KiB
    coarse, fine = _slots(sizes, 128 * 1024), _slots(sizes, 32 * 1024)
    assert coarse < fine
    imgs, refs = [], []
    for w, h in sizes:
        d = torch.full((h, w), -1, dtype=torch.int32, device=DEV)
        (x0, x1), (y0, y1) = sorted(rng.integers(0, w, 2)), sorted(rng.integers(0, h, 2))
        d[y0, x1] = d[y1, x0] = 1
        refs.append((int(x0), int(y0), int(x1 - x0 + 1), int(y1 - y0 + 1)))
        imgs.append(cmp.Image(d, d, (0, 0, w, h)))
    for slots in (coarse, fine - 1, fine):
        ws = torch.zeros(TICKETS + 16 * slots, dtype=torch.uint8, device=DEV)
        print(f"[gpu case] roi workspace of {slots} slots", flush=True)
        for _ in range(2):
            roi = cmp.roi_detect(imgs, ws=ws)
            torch.cuda.synchronize()
            assert [tuple(r) for r in roi.cpu().tolist()] == refs
    ws = torch.zeros(TICKETS + 16 * (coarse - 1), dtype=torch.uint8, device=DEV)
    with pytest.raises(cmp.CmpError) as e:   # refused on the host
        cmp.roi_detect(imgs, ws=ws)
    assert e.value.status == cmp.CMP_ENOSPC
