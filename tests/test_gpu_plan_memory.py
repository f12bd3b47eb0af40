"""The device memory of a context's launch plans is bounded: the plans used longest ago go, those of
captured calls and of kept batch sets stay.  The plan of a whole domain near 1000 x 1000 is about 90 MB,
so that 30 sizes are more than the 2 GiB that a context's plans may take."""
from __future__ import annotations

import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(300)
def test_plans_are_bounded():
    import torch
    from paper_1601_04359_amd import Context, _abi
    from test_gpu_capture import _capture

    def make(ctx, W):
        return ctx.pack(torch.from_numpy(wl.random_binary(W, W, 0.7, W)).cuda())
    with Context(0) as ctx:
        sizes = list(range(972, 1002))
        W0, W1, W2 = sizes[:3]
        out = torch.empty((1, 2 * 1002 * 1002), dtype=torch.int32, device="cuda")

        def full(bits, W, dst=None):
            dst = torch.empty((1, _abi.lpf_num_vectors(W - 1, W - 1)), dtype=torch.int32, device="cuda") \
                if dst is None else dst
            return ctx.full(bits, W, W, W - 1, W - 1, 2, out=dst)
        b0, b1, b2 = make(ctx, W0), make(ctx, W1), make(ctx, W2)
        ref0, ref1, ref2 = full(b0, W0), full(b1, W1), full(b2, W2)
        dst0 = torch.empty_like(ref0)
        graph, _ = _capture(lambda: full(b0, W0, dst0))
        set1, _, pool, descs = ctx.batch([(b1, W1, W1, W1 - 1, W1 - 1)], 2, 0)
        torch.cuda.synchronize()
        start = torch.cuda.mem_get_info()[0] + 3 * (90 << 20)
        for W in sizes[3:]:
            print(f"[gpu] plan {W}x{W}", flush=True)
            n = _abi.lpf_num_vectors(W - 1, W - 1)
            full(make(ctx, W), W, out[:, :n])
        torch.cuda.synchronize()
        used = start - torch.cuda.mem_get_info()[0]
        assert (3 << 29) < used < (2 << 30) + (128 << 20), used >> 20
        # captured: replayed with the plan it had; a batch set: the same; released: built again
        dst0.fill_(-1)
        graph.replay()
        set1.fill_(-1)
        _abi.lpf_batch(ctx.handle, pool, descs, 2, 0, set1)
        again = full(b2, W2)
        torch.cuda.synchronize()
        assert torch.equal(dst0, ref0)
        assert torch.equal(set1[:ref1.numel()].view(ref1.shape), ref1)
        assert torch.equal(again, ref2)
        del graph
