"""Limits of the over entry points on the host: what is refused does not depend
on a viewport that nothing reaches."""
import ctypes

import paper_1902_08755_amd as cmp


def test_no_layers_and_a_large_viewport():
    """Nothing to do: no tile of the viewport is counted."""
    L = cmp.lib()
    one, pitch = (ctypes.c_void_p * 1)(0x30000), (ctypes.c_int64 * 1)(8)
    for fn, extra in ((L.cmp_composite_over_backward, ()),
                      (L.cmp_composite_over_backward_as, (cmp.RGBA16F,))):
        st = fn(None, 0, cmp.RGBA32F, None, cmp.Rect(0, 0, 100000, 100000), 0x40000, 100000, one,
                *extra, pitch, None, 0, None)
        assert st == cmp.CMP_OK
