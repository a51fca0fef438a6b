"""The tiles that the autotuner times: each shape once, the defaults among them."""
import os
import re
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

TUNE = """
import ctypes, sys, torch
import paper_1902_08755_amd as cmp
dev = torch.device("cuda", 0)
for kind in (0, 1):
    shape, dtype = ((40, 600), torch.int32) if kind == 0 else ((40, 600, 4), torch.float32)
    src, out = (torch.zeros(shape, dtype=dtype, device=dev) for _ in range(2))
    depth = torch.zeros(shape, dtype=dtype, device=dev) if kind == 0 else None
    ims = cmp._images([cmp.Image(src, src if kind == 0 else None, (0, 0, 600, 40))],
                      "rgba" if kind else "u32")
    job = (cmp.CJob * 1)(cmp.CJob(kind, cmp.RGBA32F if kind else cmp.RGBA8, 1, ims,
                                  (ctypes.c_int32 * 1)(0) if kind else None,
                                  cmp.Rect(0, 0, 600, 40), out.data_ptr(),
                                  depth.data_ptr() if kind == 0 else None, 600))
    print("kind", kind, file=sys.stderr, flush=True)
    st = cmp.lib().cmp_autotune(job, 1, sys.argv[1].encode(), 1,
                                torch.cuda.current_stream().cuda_stream)
    assert st == 0, cmp.lib().cmp_last_error()
torch.cuda.synchronize()
"""


def test_autotune_times_every_shape_once(tmp_path):
    print("[gpu case] autotune candidates", flush=True)
    r = subprocess.run([sys.executable, "-c", TUNE, str(tmp_path / "cache")], cwd=ROOT, timeout=100,
                       env={**os.environ, "CMP_LOG": "1"}, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    for part, default in zip(r.stderr.split("kind 0\n")[1].split("kind 1\n"),
                             ([("64", "16")], [("128", "4"), ("256", "1")])):
        launches = re.findall(r"tiles (\d+)x(\d+), \d+ workgroups", part)
        timed = launches[::2]   # a launch to warm up, then one to time
        assert timed == launches[1::2] and len(set(timed)) == len(timed) > 4, timed
        assert all(d in timed for d in default)
