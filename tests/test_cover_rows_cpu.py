"""Launch plans of lpf_full run on the host with the kernel's own index arithmetic, for images of a
few long rows: 64 lanes per row, so that a tile is as many rows as the image has, down to one."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl


@pytest.mark.parametrize("W,H,cx,cy", [(1025, 1, 1024, 0), (1040, 1, 300, 0), (1500, 1, 600, 0),
                                       (2048, 1, 500, 0), (4000, 1, 1000, 0), (2048, 2, 400, 1),
                                       (3000, 2, 300, 0), (2049, 3, 260, 2)])
def test_few_long_rows(W, H, cx, cy):
    from paper_1601_04359_amd import _abi
    img = np.ones((H, W), np.uint8)  # runs longer than the cutoff, and short ones
    img[:, W // 5] = 0
    img[H // 2, W // 2: W // 2 + 200] = wl.random_binary(200, 1, 0.8, W)[0]
    ref = oracle.lpf(img, cx, cy, 3)
    for phase in (0, 1):
        got = _abi.lpf_cover_counts(img, cx, cy, phase)
        assert np.array_equal(got, ref[phase]), int((got != ref[phase]).sum())
