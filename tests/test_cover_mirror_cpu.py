"""Launch plans of lpf_full whose groups of both signs of dx share words and records: where the axis
(the paths of dx = 0 or dy = 0, which have no mirrored image) is a part of a group, several groups, or
a group apart from the others."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl


# the axis within a group; it alone in its groups and a part of the next; paths of one octant only;
# all paths in one group; the axis apart (many members in few groups)
@pytest.mark.parametrize("W,H,cx,cy,shape", [(33, 50, 7, 9, (0, 0, 0, 0)), (400, 12, 399, 11, (0, 0, 0, 0)),
                                             (5, 1300, 4, 1200, (0, 0, 0, 0)), (60, 40, 30, 1, (0, 0, 0, 0)),
                                             (40, 60, 0, 30, (0, 0, 0, 0)), (64, 64, 2, 2, (0, 0, 0, 0)),
                                             (400, 90, 399, 89, (1, 1, 0, 0))])
def test_mirrored_groups(W, H, cx, cy, shape):
    from paper_1601_04359_amd import _abi
    img = wl.boolean_disks(W, H, min(W, H) / 4.0, 0.95, W + H)
    img[:, W // 3:] |= 1  # long runs
    img[H // 2, W // 2] = img[H // 4, W // 8] = 0
    got = _abi.lpf_cover_counts(img, cx, cy, 1, *shape)
    v = oracle.vectors(cx, cy)
    idx = np.unique(np.concatenate([np.arange(0, len(v), 1 + len(v) // 500), np.flatnonzero((v == 0).any(1)),
                                    np.flatnonzero(np.abs(v[:, 0]) == np.abs(v[:, 1]))]))
    assert np.array_equal(got[idx], oracle.lpf_vectors(img, v[idx], 2)[0])
