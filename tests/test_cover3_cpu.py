"""Launch plans of lpf_full3d run on the host (lpf_cover3_counts) against the oracle: every count,
with every LDS access of the plan checked."""
from __future__ import annotations

import numpy as np
import pytest

import oracle

# rows of one to four words and of several strips, partial words, slabs of all planes and of one or
# two, degenerate axes, cuts (cz = 0), the largest cutoff
CASES = [(1, 1, 1, 0, 0, 0), (5, 4, 3, 4, 3, 2), (33, 9, 7, 6, 8, 5), (64, 20, 12, 7, 5, 11),
         (96, 11, 9, 3, 4, 2), (100, 13, 10, 6, 6, 6), (130, 7, 6, 5, 3, 2), (40, 36, 35, 0, 9, 0),
         (40, 36, 5, 24, 0, 3), (60, 200, 30, 5, 4, 6), (34, 34, 3, 25, 2, 1)]


@pytest.mark.parametrize("W,H,D,cx,cy,cz", CASES)
def test_plan_counts_equal_oracle(W, H, D, cx, cy, cz):
    from paper_1601_04359_amd import _abi
    g = np.random.default_rng(W * 100 + H)
    vol = (g.random((D, H, W)) < 0.85).astype(np.uint8)
    vol[:, : H // 2] = 1  # long segments survive there, and end everywhere else
    vol[0, 0, 0] = 0
    if cx > 24:
        with pytest.raises(_abi.LpfError) as e:
            _abi.lpf_cover3_counts(vol, cx, cy, cz, 1)
        assert e.value.status == _abi.LPF_E_UNSUPPORTED
        return
    ref = oracle.lpf3(vol, cx, cy, cz, 3)
    for phase in (0, 1):
        got = _abi.lpf_cover3_counts(vol, cx, cy, cz, phase)
        assert np.array_equal(got, ref[phase]), int((got != ref[phase]).sum())
