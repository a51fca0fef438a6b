"""Argument checks of the adjoint with a chosen gradient type: refused on the
host before anything is enqueued."""
import ctypes

import pytest

import paper_1902_08755_amd as cmp


@pytest.mark.parametrize("grad_fmt,ptr,pitch,grad_out,ok", [
    (cmp.RGBA16F, 0x30004, 8, 0x40000, False),   # halves need 8-byte alignment
    (cmp.RGBA32F, 0x30008, 8, 0x40000, False),   # floats 16
    (cmp.RGBA8, 0x30000, 8, 0x40000, False),     # not a float format
    (7, 0x30000, 8, 0x40000, False),
    (cmp.RGBA16F, 0x30008, 7, 0x40000, False),   # pitch below the ROI's width
    (cmp.RGBA16F, 0, 8, 0x40000, False),
    (cmp.RGBA16F, 0x30008, 8, 0x40008, False),   # the incoming gradient is FP32
    (cmp.RGBA16F, 0x30008, 8, 0, False),
    (cmp.RGBA16F, 0x30008, 8, 0, True)])         # nothing to do: no layers
def test_backward_as_argument_errors(grad_fmt, ptr, pitch, grad_out, ok):
    L = cmp.lib()
    n = 0 if ok else 2
    arr = (cmp.CImage * 2)(*[cmp.CImage(0x10000, None, 8, cmp.Rect(0, 0, 8, 8))] * 2)
    gl, gp = (ctypes.c_void_p * 2)(0x30000, ptr), (ctypes.c_int64 * 2)(8, pitch)
    st = L.cmp_composite_over_backward_as(arr, n, cmp.RGBA32F, (ctypes.c_int32 * 2)(1, 0),
                                          cmp.Rect(0, 0, 8, 8), grad_out, 8, gl, grad_fmt, gp,
                                          None, 0, None)
    assert st == (cmp.CMP_OK if ok else cmp.CMP_EINVAL)
