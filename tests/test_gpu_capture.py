"""Calls captured in a graph stay right when later calls of the same context use more scratch, other
plans and other batches: the memory that a captured call reads is kept.  Whole numbers, every replay
against the eager result, with the program's own eager work between the replays."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


def _capture(f):
    """f captured on a stream of its own, after two calls outside the capture; (graph, outputs)."""
    import torch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        for _ in range(2):
            f()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        out = f()
    return g, out


def _replays(g, out, ref, between, n=3):
    import torch
    for i in range(n):
        between(i)
        torch.cuda.synchronize()
        out.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref), i


def _junk():
    """Allocations that take the place of what the context has freed."""
    import torch
    for mb in (1, 2, 8, 32, 64):
        torch.full((mb << 18,), -1, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def test_delta_scratch_stays():
    import torch
    from paper_1601_04359_amd import Context
    W, H, c = 128, 96, 20
    img = wl.boolean_disks(W, H, 6.0, 0.5, 3)
    ones, zeros = np.flatnonzero(img == 1), np.flatnonzero(img == 0)
    g = np.random.default_rng(1)

    def swaps(n):
        return torch.from_numpy(np.stack([g.choice(ones, n), g.choice(zeros, n)], 1).astype(np.int32)).cuda()
    print("[gpu] capture delta", flush=True)
    with Context(0) as ctx:
        bits = ctx.pack(torch.from_numpy(img).cuda())
        few, many = swaps(40), swaps(9000)
        ref = ctx.delta_swap(bits, W, H, c, c, few)
        graph, out = _capture(lambda: ctx.delta_swap(bits, W, H, c, c, few))

        def between(i):
            ctx.delta_swap(bits, W, H, c + i, c, many)
            torch.cuda.synchronize()
            _junk()
        _replays(graph, out, ref, between)
        del graph
