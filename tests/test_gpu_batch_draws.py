"""Batches of more items than workgroups, whose workgroups draw from the queues,
take from each other's and reset them for the next launch: counts just above
the number of workgroups, and one costly job among many cheap ones. Every job
against its plain call, bit for bit, in replays without an upload in between."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1902_08755_amd as cmp
from test_gpu_batch_queues import DEV, _job

pytestmark = pytest.mark.gpu


def _batch(jobs):
    arr, outs, keep = (cmp.CJob * len(jobs))(), [], []
    for k, (kind, w, h, imgs, order) in enumerate(jobs):
        ims = cmp._images(imgs, "rgba" if kind else "u32")
        o = (ctypes.c_int32 * len(order))(*order)
        if kind:
            out = (torch.zeros((h, w, 4), device=DEV),)
        else:
            out = tuple(torch.zeros((h, w), dtype=torch.int32, device=DEV) for _ in range(2))
        arr[k] = cmp.CJob(kind, cmp.RGBA32F if kind else cmp.RGBA8, len(imgs), ims,
                          o if kind else None, cmp.Rect(0, 0, w, h), out[0].data_ptr(),
                          None if kind else out[1].data_ptr(), w)
        outs.append(out)
        keep += [ims, o]
    plan = ctypes.c_void_p()
    assert cmp.lib().cmp_batch_plan_create(arr, len(jobs), None, ctypes.byref(plan)) == 0
    items, workgroups = ctypes.c_int64(), ctypes.c_int32()
    assert cmp.lib().cmp_batch_info(plan, ctypes.byref(items), ctypes.byref(workgroups)) == 0
    return plan, outs, keep, items.value, workgroups.value


def _workgroups():
    plan, _, _, _, workgroups = _batch([_job(np.random.default_rng(0), 0, 4, 4, 1)])
    cmp.lib().cmp_batch_plan_destroy(plan)
    return workgroups


@pytest.mark.parametrize("case", ["one more", "33 more", "costly over", "costly depth",
                                  "two costly"])
def test_batch_draws(case):
    rng = np.random.default_rng(len(case))
    if case.endswith("more"):   # jobs of one tile each
        n = _workgroups() // 32 * 32 + (1 if case == "one more" else 33)
        jobs = [_job(rng, k % 2, 20, 3, 1 + k % 3) for k in range(n)]
    else:
        jobs = [_job(rng, k % 2, int(rng.integers(1, 90)), int(rng.integers(1, 70)), 1 + k % 4)
                for k in range(61)]
        if case != "costly depth":
            jobs.insert(30, _job(rng, 1, 1100, 1021, 12))
        if case != "costly over":
            jobs.insert(11, _job(rng, 0, 1700, 1303, 45))
    plan, outs, keep, items, workgroups = _batch(jobs)
    print(f"[gpu case] batch draws, {case}: {items} items, {workgroups} workgroups", flush=True)
    # (up to as many items as workgroups, in whole groups of 32, none is drawn)
    assert items == n if case.endswith("more") else items > workgroups
    L, s = cmp.lib(), torch.cuda.current_stream().cuda_stream
    ws = torch.zeros(L.cmp_batch_workspace_size(plan), dtype=torch.uint8, device=DEV)
    assert L.cmp_batch_upload(plan, ws.data_ptr(), ws.numel(), s) == 0
    torch.cuda.synchronize()
    assert L.cmp_batch_run_plain(plan, s) == 0
    want = [tuple(t.clone() for t in out) for out in outs]
    for _ in range(4):
        for out in outs:
            for t in out:
                t.fill_(7)
        assert L.cmp_batch_run(plan, ws.data_ptr(), s) == 0
        torch.cuda.synchronize()
        assert all(torch.equal(t, r) for out, ref in zip(outs, want) for t, r in zip(out, ref))
    # back to back, without a host wait between
    for _ in range(5):
        assert L.cmp_batch_run(plan, ws.data_ptr(), s) == 0
    torch.cuda.synchronize()
    assert all(torch.equal(t, r) for out, ref in zip(outs, want) for t, r in zip(out, ref))
    L.cmp_batch_plan_destroy(plan)
    del keep
