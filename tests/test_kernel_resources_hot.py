"""The waves per SIMD (workgroups per compute unit) that the kernels of the main
path are measured at, and no scratch memory in any kernel: closer bounds than
the general ones, over every instance."""
import re

import pytest

from test_kernel_resources import usage  # noqa: F401 (the fixture)

# by kernel name: every instance of a template is held to it
WAVES = {
    "roi_kernel": 8, "depth_kernel": 8, "depth_small_kernel": 8,
    "rle_compress_kernel": 4, "rle_decompress_kernel": 5,
    "rle64_compress_kernel": 4, "rle64_decompress_kernel": 3,
    "over_kernel": 6, "over_tree_kernel": 7, "over_bwd_kernel": 2, "batch_kernel": 6,
}


def test_no_kernel_uses_scratch_memory(usage):  # noqa: F811
    assert {name: u["ScratchSize"] for name, u in usage.items() if u["ScratchSize"]} == {}


@pytest.mark.parametrize("kernel", list(WAVES))
def test_waves_per_simd(usage, kernel):  # noqa: F811
    # mangled in the namespace: _ZN3cmp<length><name>...
    found = {n: u for n, u in usage.items()
             if re.match(rf"_ZN3cmp{len(kernel)}{kernel}(?![a-z0-9_])", n)}
    assert found
    for name, u in found.items():
        assert u["Occupancy"] >= WAVES[kernel], (name, u)
        assert u["LDS Size"] * WAVES[kernel] <= 160 * 1024, (name, u)
