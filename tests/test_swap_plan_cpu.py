"""Launch plans of lpf_delta_swap run on the host (lpf_swap_plan_delta) against the oracle: every
change, with every table entry checked against its array."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl

# windows wider than the cell (periodic images of the changed pixels), degenerate cutoffs,
# paths of 1 to 127 pixels
CASES = [(1, 1, 0, 0), (5, 3, 4, 2), (9, 7, 8, 6), (40, 3, 39, 0), (2, 40, 1, 39), (30, 21, 12, 20),
         (70, 66, 48, 47), (66, 66, 63, 63), (70, 70, 64, 12), (130, 9, 126, 8), (9, 129, 5, 126)]


@pytest.mark.parametrize("W,H,cx,cy", CASES)
def test_plan_changes_equal_oracle(W, H, cx, cy):
    from paper_1601_04359_amd import _abi
    img = (wl.random_binary(W, H, 0.8, 7 * W + H) | wl.stripes(W, H, 16, 5)).astype(np.uint8)
    img.flat[0], img.flat[-1] = 1, 0
    if W * H == 1:
        with pytest.raises(_abi.LpfError):  # no interchange
            _abi.lpf_swap_plan_delta(img, cx, cy, 0, 0)
        return
    g = np.random.default_rng(W + H)
    ones, zeros = np.flatnonzero(img == 1), np.flatnonzero(img == 0)
    swaps = [(0, W * H - 1)] + [(int(g.choice(ones)), int(g.choice(zeros))) for _ in range(3)]
    ref = oracle.delta_swap(img, cx, cy, np.array(swaps, np.int32), 3)
    for i, (a, b) in enumerate(swaps):
        assert np.array_equal(_abi.lpf_swap_plan_delta(img, cx, cy, a, b), ref[i])


def test_plan_refuses_large_cutoffs():
    from paper_1601_04359_amd import _abi
    img = wl.stripes(140, 4, 16, 5).astype(np.uint8)
    a, b = int(np.flatnonzero(img == 1)[0]), int(np.flatnonzero(img == 0)[0])
    with pytest.raises(_abi.LpfError) as e:
        _abi.lpf_swap_plan_delta(img, 127, 2, a, b)
    assert e.value.status == _abi.LPF_E_UNSUPPORTED
