"""Launch plans of lpf_full run on the host (lpf_cover_counts) against the oracle: every count, with
every LDS access of the plan checked against its array."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl

# W, H, cutoff x, cutoff y, forced (R, S, waves, LDS bytes): lanes of 1..16 words, several lanes
# per row, several tiles down and across, partial last words and bands, rows narrower than a word,
# the whole domain, degenerate domains, one-mask plans of a small staging budget
CASES = [
    (64, 64, 16, 16, (0, 0, 0, 0)),
    (1, 1, 0, 0, (0, 0, 0, 0)),
    (5, 3, 4, 2, (0, 0, 0, 0)),
    (33, 50, 0, 20, (0, 0, 0, 0)),
    (33, 50, 20, 0, (0, 0, 0, 0)),
    (40, 37, 39, 36, (0, 0, 0, 0)),
    (31, 130, 12, 65, (0, 0, 0, 0)),
    (97, 65, 30, 31, (0, 0, 0, 0)),
    (333, 70, 40, 21, (0, 0, 0, 0)),
    (530, 20, 25, 19, (0, 0, 0, 0)),
    (700, 9, 16, 8, (0, 0, 0, 0)),
    (100, 300, 20, 60, (0, 0, 0, 8192)),
    (200, 150, 20, 17, (1, 8, 0, 0)),
    (200, 150, 20, 17, (4, 2, 2, 8192)),
    (200, 150, 20, 17, (2, 0, 4, 0)),
    (200, 150, 20, 17, (1, 0, 1, 0)),
    (200, 90, 30, 30, (8, 4, 3, 0)),
]


@pytest.mark.parametrize("W,H,cx,cy,shape", CASES)
def test_plan_counts_equal_oracle(W, H, cx, cy, shape):
    from paper_1601_04359_amd import _abi
    # dense in phase 1 (long segments survive) with a random part
    img = (wl.random_binary(W, H, 0.9, 7 * W + H) | wl.stripes(W, H, 16, 5)).astype(np.uint8)
    ref = oracle.lpf(img, cx, cy, 3)
    for phase in (0, 1):
        got = _abi.lpf_cover_counts(img, cx, cy, phase, *shape)
        assert np.array_equal(got, ref[phase]), int((got != ref[phase]).sum())


@pytest.mark.parametrize("c", [128, 200])
def test_plan_of_large_cutoffs(c):
    # many groups, long words, paths cut into several walks (axes and diagonals)
    from paper_1601_04359_amd import _abi
    img = wl.boolean_disks(c + 1, c + 1, 30.0, 0.9, 3)
    got = _abi.lpf_cover_counts(img, c, c, 1)
    v = oracle.vectors(c, c)
    idx = np.unique(np.concatenate([np.arange(0, len(v), 37), np.flatnonzero(np.abs(v).max(1) == c)[::9]]))
    assert np.array_equal(got[idx], oracle.lpf_vectors(img, v[idx], 2)[0])


def test_plan_refuses_rows_that_do_not_fit():
    from paper_1601_04359_amd import _abi
    with pytest.raises(_abi.LpfError) as e:
        _abi.lpf_cover_counts(wl.random_binary(64, 64, 0.5, 1), 16, 16, 1, 0, 0, 0, 1)
    assert e.value.status == _abi.LPF_E_UNSUPPORTED
