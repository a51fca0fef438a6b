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


@pytest.mark.parametrize("types", [[torch.bfloat16], [torch.float64], [torch.bfloat16] * 3,
                                   [torch.float32, torch.float16], [torch.float16, torch.float32],
                                   [torch.float32, torch.float64], [torch.int32]])
def test_gradient_types(types):
    """Gradients that the kernel would write past the end of, or as other numbers."""
    layers = [cmp.Image(_empty(), None, (0, 0, 7, 0)) for _ in types]
    grads = [torch.zeros((2, 7, 4), dtype=t) for t in types]
    with pytest.raises(ValueError, match="all float32 or all float16"):
        cmp.composite_over_backward(layers, list(range(len(types))), (0, 0, 7, 2),
                                    torch.zeros((2, 7, 4)), grads=grads)


@pytest.mark.parametrize("first,other", [(torch.float32, torch.float16),
                                         (torch.float16, torch.float32),
                                         (torch.float16, torch.bfloat16)])
def test_layers_of_several_types(first, other):
    """One pixel format per call: a layer of another type would be read as the
    first one's, out of range where its pixels are smaller."""
    rois, order, vp = [(0, 0, 7, 0), (0, 0, 7, 2)], [1, 0], (0, 0, 7, 2)
    pixels = [_empty(first), torch.zeros((2, 7, 4), dtype=other)]
    layers = [cmp.Image(t, None, r) for t, r in zip(pixels, rois)]
    out, match = torch.zeros((2, 7, 4)), f"expected {first} pixels, got {other}"
    with pytest.raises(ValueError, match=match):
        cmp.composite_over(layers, order, vp, out=out)
    with pytest.raises(ValueError, match=match):
        cmp.composite_over_backward(layers, order, vp, out)
    with pytest.raises(ValueError, match=match):
        cmp.OverComposite.apply(order, vp, rois, *pixels)
    # a layer that covers nothing is not read: refused for its device only
    with pytest.raises(ValueError, match="device tensor"):
        cmp.composite_over([layers[0], cmp.Image(pixels[1], None, (0, 0, 0, 0))], order, vp,
                           out=out)


@pytest.mark.parametrize("fmt,dtype", [(cmp.RGBA32F, torch.float16), (cmp.RGBA32F, torch.int16),
                                       (cmp.RGBA16F, torch.float32), (cmp.RGBA16F, torch.uint8)])
def test_roi_pixels_of_the_format(fmt, dtype):
    """Float images whose pixels are not the size of the format's."""
    imgs = [cmp.Image(_empty(), None, (0, 0, 7, 0)),
            cmp.Image(torch.zeros((2, 7, 4), dtype=dtype), None, (0, 0, 7, 2))]
    with pytest.raises(ValueError, match="expected pixels of"):
        cmp.roi_detect(imgs, fmt=fmt)
    with pytest.raises(ValueError, match="expected pixels of"):
        cmp.roi_grid(imgs, (4, 4), fmt=fmt)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float64])
def test_composite_and_its_gradient_are_float32(dtype):
    """The composite is written, and its gradient read, at 16 bytes per pixel."""
    layers, vp = [cmp.Image(_empty(), None, (0, 0, 7, 0))], (0, 0, 7, 2)
    other = torch.zeros((2, 7, 4), dtype=dtype)
    with pytest.raises(ValueError, match="out must hold float32"):
        cmp.composite_over(layers, [0], vp, out=other)
    with pytest.raises(ValueError, match="grad_out must hold float32"):
        cmp.composite_over_backward(layers, [0], vp, other)


def test_workspaces_kept():
    """A bounded number, the least recently used given back; grown on demand."""
    first = cmp.workspace("kept", 100, "cpu")
    assert first.numel() >= 100 and not bool(first.any())
    assert cmp.workspace("kept", 50, "cpu") is first
    for k in range(200):
        cmp.workspace(f"kept {k}", 8, "cpu")
        assert cmp.workspace("kept", 100, "cpu") is first
    assert len(cmp._workspaces) <= 64
    assert cmp.workspace("kept", 1000, "cpu").numel() >= 1000
    cmp._workspaces.clear()
