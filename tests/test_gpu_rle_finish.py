"""The end of a compression, where its workgroups are counted one by one (few of
them, or many slots each) or in groups: calls of both kinds in turn on one
workspace, each repeated, leave it ready for the next."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_08755_amd as cmp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _images(rng, sizes):
    out = []
    for w, h in sizes:
        t = [torch.from_numpy(np.repeat(rng.integers(0, 1 << 31, size=(h, (w + 3) // 4)), 4, axis=1)
                              [:, :w].astype(np.int32)).to(DEV) for _ in range(2)]
        out.append(cmp.Image(t[0], t[1], (0, 0, w, h)))
    return out


@pytest.mark.parametrize("codec", ["rle", "rle64"])
def test_counts_in_turn(codec):
    rng = np.random.default_rng(9)
    # slots: 1, 64 (as many as are counted one by one), 130, about 900, about
    # 1500 and about 2500 (a device holds about 1000 workgroups)
    sets = [_images(rng, s) for s in ([(9, 9)], [(64, 64)] * 64, [(512, 1040)],
                                      [(700, 750)] * 7, [(1024, 1000)] * 6, [(2000, 1700)] * 3)]
    want = []
    for imgs in sets:
        f = oracle.rle_compress if codec == "rle" else oracle.rle64_compress
        want.append([f(i.color.cpu().numpy().view(np.uint32), i.depth.cpu().numpy().view(np.uint32),
                       i.roi) for i in imgs[:2]])
    ws = torch.zeros(max(int(cmp.lib().cmp_rle_workspace_size(cmp._images(i, "u32"), len(i)))
                         for i in sets), dtype=torch.uint8, device=DEV)
    batches = [cmp.RleBatch(i) for i in sets]
    for b in batches:
        b.ws = ws
    for k in [0, 3, 3, 5, 4, 4, 1, 2, 5, 3, 0, 4, 2, 2, 1, 5, 3]:
        print(f"[gpu case] rle finish {codec} set {k}", flush=True)
        if codec == "rle":
            for t in batches[k].outs:
                t.zero_()
            streams, sizes, status = batches[k].run()
        else:
            streams, sizes, status = cmp.rle64_compress(sets[k])
        assert int(status.abs().sum()) == 0
        for s, n, ref in zip(streams, sizes.tolist(), want[k]):
            assert n == ref.size and (s[:n].cpu().numpy() == ref).all()
