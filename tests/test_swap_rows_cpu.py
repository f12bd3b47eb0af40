"""The words that lpf_delta_swap takes from packed rows, by its launch plan's host run (which sets the
bits past the row's width: they are no part of the image): cells narrower than a word, whose row
repeats within it, and widths around one and two words."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl


@pytest.mark.parametrize("W", [1, 2, 3, 7, 15, 16, 17, 20, 30, 31, 32, 33, 45, 63, 64, 65, 96, 97])
def test_rows_ignore_their_padding(W):
    from paper_1601_04359_amd import _abi
    H, cx, cy = 9, min(W - 1, 18), 6
    img = (wl.random_binary(W, H, 0.8, W) | wl.stripes(W, H, 16, 5)).astype(np.uint8)
    img.flat[0], img.flat[-1] = 1, 0
    ones, zeros = np.flatnonzero(img == 1), np.flatnonzero(img == 0)
    g = np.random.default_rng(W)
    swaps = [(int(g.choice(ones)), int(g.choice(zeros))) for _ in range(4)]
    ref = oracle.delta_swap(img, cx, cy, np.array(swaps, np.int32), 3)
    for (a, b), r in zip(swaps, ref):
        assert np.array_equal(_abi.lpf_swap_plan_delta(img, cx, cy, a, b), r)
