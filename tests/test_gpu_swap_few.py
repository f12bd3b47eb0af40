"""lpf_delta_swap with a few vectors and many candidates, on both sides of the lines between offset rows
and shared segments (16384 candidates up to 26 changes each, 49152 up to 36), against the oracle.
Whole numbers."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_delta import _gpu_delta, _swaps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,cx,cy,mask,n", [
    (9, 7, 0, 0, 3, 16385), (40, 33, 2, 2, 3, 16384), (40, 33, 2, 2, 3, 16385), (20, 70, 0, 5, 3, 40000),
    (33, 9, 3, 3, 2, 17000), (33, 9, 3, 3, 3, 50000), (70, 20, 6, 0, 1, 17000), (16, 40, 2, 3, 3, 49152),
    (16, 40, 2, 3, 3, 49153)])
def test_few_vectors(W, H, cx, cy, mask, n):
    import torch
    from paper_1601_04359_amd import Context
    print(f"[gpu] swap {W}x{H} c=({cx},{cy}) mask={mask} n={n}", flush=True)
    img = wl.boolean_disks(W, H, 3.0, 0.5, W)
    sw = _swaps(img, n, 8, near=6)
    with Context(0) as ctx:
        got = _gpu_delta(ctx, img, cx, cy, sw, mask)
        torch.cuda.synchronize()
    i = np.unique(np.concatenate([np.arange(0, n, 61), np.arange(n - 300, n)]))
    assert np.array_equal(got[i], oracle.delta_swap(img, cx, cy, sw[i], mask))
