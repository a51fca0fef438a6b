"""What the Python binding accepts and refuses before it reaches the device."""
import numpy as np
import pytest
import torch

import paper_1902_08755_amd as cmp


def _empty(dtype=torch.float32):
    """A layer without pixels: packed without a look at its device."""
    return torch.zeros((0, 7, 4), dtype=dtype)


@pytest.mark.parametrize("roi", [torch.tensor([1.0, 2.5, 5.0, 0.0]),
                                 [torch.tensor(v) for v in (1.0, 2.5, 5.0, 0.0)],
                                 [np.array(v) for v in (1.0, 2.5, 5.0, 0.0)],
                                 np.array([1.0, 2.5, 5.0, 0.0]), ("1", "2", "5", "0")])
def test_rectangles_of_other_numbers(roi):
    """Whatever int() takes is a coordinate, as in one ctypes object per rectangle."""
    arr = cmp._images([cmp.Image(_empty(), None, (9, 8, 7, 0)), cmp.Image(_empty(), None, roi)],
                      "rgba")
    want = [(9, 8, 7, 0), tuple(int(v) for v in roi)]
    assert [(a.roi.x, a.roi.y, a.roi.w, a.roi.h) for a in arr] == want
    assert [a.pitch for a in arr] == [7, 5]
