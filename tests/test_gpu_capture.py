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


def test_batch_tables_stay():
    # more sets than the context keeps, and images with rows in device memory of growing sizes
    import torch
    from paper_1601_04359_amd import Context, _abi
    print("[gpu] capture batch", flush=True)
    with Context(0) as ctx:
        def items(k):
            sizes = [(48 + k, 40, 12, 10), (64, 33 + k, 20, 16), (70 + 60 * k, 50 + 40 * k, 9, 9)]
            return [(ctx.pack(torch.from_numpy(wl.random_binary(W, H, 0.7, W + H)).cuda()), W, H, cx, cy)
                    for W, H, cx, cy in sizes]
        for lds in (0, 1):  # staged in LDS, in device memory
            ctx.set_full_shape(0, 0, 0, lds)
            first = items(0)
            ref, offs, pool, descs = ctx.batch(first, 3, 0)
            counts = torch.empty_like(ref)

            def call():
                _abi.lpf_batch(ctx.handle, pool, descs, 3, 0, counts)
                return counts
            graph, out = _capture(call)

            def between(i):
                for k in range(1 + 9 * i, 10 + 9 * i):
                    ctx.batch(items(k), 3, 0)
                torch.cuda.synchronize()
                _junk()
            _replays(graph, out, ref, between)
            del graph
