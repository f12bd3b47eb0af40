"""lpf_full3d by prefix trees at the edges of its launches: rows of one to four words and of several
strips, one and several slabs, single phases, and the volumes that keep the voxel-by-voxel kernels.
Whole numbers, no tolerance."""
from __future__ import annotations

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,D,cx,cy,cz,mask", [
    (1, 1, 1, 0, 0, 0, 3), (20, 9, 7, 6, 8, 5, 3), (33, 70, 40, 4, 6, 9, 2), (64, 20, 12, 7, 5, 11, 1),
    (90, 40, 60, 5, 4, 3, 3), (120, 33, 50, 8, 8, 8, 3), (260, 21, 9, 3, 4, 2, 3),
    (40, 36, 5, 24, 0, 3, 3), (60, 200, 90, 2, 3, 20, 3), (40, 36, 5, 25, 2, 3, 3), (520, 9, 8, 2, 2, 2, 3)])
def test_counts_equal_oracle(W, H, D, cx, cy, cz, mask):
    import torch
    from paper_1601_04359_amd import Context
    print(f"[gpu] volume {W}x{H}x{D} c=({cx},{cy},{cz}) mask={mask}", flush=True)
    g = np.random.default_rng(W + H + D)
    vol = (g.random((D, H, W)) < 0.7).astype(np.uint8)
    vol[:, : H // 2] = 1
    vol[0, 0, 0] = 0
    with Context(0) as ctx:
        bits = ctx.pack3d(torch.from_numpy(vol).cuda())
        ref = oracle.lpf3(vol, cx, cy, cz, mask)
        for _ in range(2):
            got = ctx.full3d(bits, W, H, D, cx, cy, cz, mask).cpu().numpy()
            assert np.array_equal(got, ref)
