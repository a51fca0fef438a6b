"""A view one pixel wide, of so many rows that the shape which a requested tile
is run as has to be made higher to stay within the tiles of a launch."""
import pytest
import torch

import paper_1902_08755_amd as cmp

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def test_over_tall_and_narrow():
    h = (1 << 26) + 5   # 16x16 runs as 64x4: 2^24 + 2 tiles
    layer = torch.randint(0, 1 << 14, (h, 1, 4), dtype=torch.int16, device=DEV).view(torch.float16)
    out = torch.full((h, 1, 4), 7., device=DEV)
    print(f"[gpu case] over 1x{h}, tiles of 16x16", flush=True)
    cmp.composite_over([cmp.Image(layer, None, (0, 0, 1, h))], [0], (0, 0, 1, h), out=out,
                       tile=(16, 16))
    torch.cuda.synchronize()
    assert torch.equal(out.half(), layer)   # one layer over nothing is the layer
