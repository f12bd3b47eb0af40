"""What lpf_autotune_full records is the cover kernel's: the calls that walk chains (no allocation,
rows in device memory) keep their own shapes, and every call that ran before tuning runs after it."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def _tuned(ctx, W, H, cx, cy):
    import torch
    print(f"[gpu] tuned {W}x{H} cutoff ({cx}, {cy})", flush=True)
    bits = ctx.pack(torch.from_numpy(wl.boolean_disks(W, H, 5.0, 0.5, W)).cuda())
    ref = ctx.full(bits, W, H, cx, cy)
    assert ctx.autotune(bits, W, H, cx, cy) > 0
    print(f"[gpu] shape {ctx.tuned_shape(W, H, cx, cy)}", flush=True)
    assert torch.equal(ctx.full(bits, W, H, cx, cy), ref)
    return bits, ref


# automatic lanes of 3, 4, 7, 11 and 12 words
@pytest.mark.parametrize("W,H,cx,cy", [(96, 64, 16, 16), (100, 300, 20, 40), (200, 90, 20, 20),
                                       (333, 100, 30, 20), (384, 200, 60, 60)])
def test_chain_walks_after_tuning(W, H, cx, cy):
    import torch
    from paper_1601_04359_amd import Context, _abi
    with Context(0) as ctx:
        bits, ref = _tuned(ctx, W, H, cx, cy)
        got = torch.empty_like(ref)
        _abi.lpf_full_noalloc(ctx.handle, bits, W, H, cx, cy, 3, 0, got)
        assert torch.equal(got, ref)
        ctx.set_full_shape(0, 0, 0, 1)  # rows in device memory
        assert torch.equal(ctx.full(bits, W, H, cx, cy), ref)


# 8224 x 2300: rows fit LDS with 4 words per lane only, in 65 tiles across; a fixed R of 4 would need
# more than 64 lanes per row
@pytest.mark.parametrize("W,H,cx,cy", [(96, 64, 16, 16), (256, 90, 30, 30), (333, 100, 30, 20),
                                       (700, 60, 20, 20), (8224, 2300, 1, 2250)])
def test_recorded_shape_is_accepted(W, H, cx, cy):
    import torch
    from paper_1601_04359_amd import Context
    with Context(0) as ctx:
        bits, ref = _tuned(ctx, W, H, cx, cy)
        counts, _, _, _ = ctx.batch([(bits, W, H, cx, cy)], 3, 0)
        assert torch.equal(counts[:ref.numel()].view(ref.shape), ref)
        R, wpg, lds = ctx.tuned_shape(W, H, cx, cy)
        ctx.set_full_shape(R, 0, wpg, lds)
        assert torch.equal(ctx.full(bits, W, H, cx, cy), ref)


def test_losing_plans_are_released():
    # 512^2, cutoff 255: a plan is about 8 MB, the autotuner makes up to 21 of them
    import torch
    from paper_1601_04359_amd import Context
    W, c = 512, 255
    with Context(0) as ctx:
        bits = ctx.pack(torch.from_numpy(wl.boolean_disks(W, W, 9.0, 0.5, 1)).cuda())
        ref = ctx.full(bits, W, W, c, c)
        print("[gpu] tuned: memory", flush=True)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        for _ in range(2):
            ctx.autotune(bits, W, W, c, c)
            assert torch.equal(ctx.full(bits, W, W, c, c), ref)
        torch.cuda.synchronize()
        # the plan from before, the chosen one, chain tables of shapes that do not fit LDS
        assert before - torch.cuda.mem_get_info()[0] < 40 << 20
