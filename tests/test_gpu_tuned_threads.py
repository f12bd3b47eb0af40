"""A batch of the image size that another thread tunes: the set that it keeps goes on reading the plan
that it was made with, also where that plan lost."""
from __future__ import annotations

import threading

import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def test_batch_sets_while_tuning():
    import torch
    from paper_1601_04359_amd import Context, _abi
    W, H, c = 400, 300, 60
    with Context(0) as ctx:
        bits = ctx.pack(torch.from_numpy(wl.boolean_disks(W, H, 9.0, 0.5, 5)).cuda())
        ref = ctx.full(bits, W, H, c, c)
        counts, _, pool, descs = ctx.batch([(bits, W, H, c, c)], 3, 0)
        torch.cuda.synchronize()
        wrong, calls, done = [], [0], threading.Event()

        def batches():
            with torch.cuda.stream(torch.cuda.Stream()):
                out = torch.empty_like(counts)
                while not done.is_set() and calls[0] < 2000:
                    out.fill_(-1)
                    _abi.lpf_batch(ctx.handle, pool, descs, 3, 0, out)
                    if not torch.equal(out[:ref.numel()].view(ref.shape), ref):
                        wrong.append(calls[0])
                    calls[0] += 1
        print(f"[gpu] batch and tuning at once {W}x{H}", flush=True)
        th = threading.Thread(target=batches)
        th.start()
        try:
            for _ in range(2):
                assert ctx.autotune(bits, W, H, c, c) > 0
        finally:
            done.set()
            th.join()
        print(f"[gpu] {calls[0]} batches", flush=True)
        assert calls[0] and not wrong
        for _ in range(2):
            counts.fill_(-1)
            _abi.lpf_batch(ctx.handle, pool, descs, 3, 0, counts)
            assert torch.equal(counts[:ref.numel()].view(ref.shape), ref)
