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
