"""lpf_delta_swap by shared segments at the edges of its launches: partial words of 32 candidates,
several scratch batches, one and several sectors, single phases, against the oracle or (many
candidates) the run-based kernel.  Whole numbers, no tolerance."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl
from test_gpu_delta import _gpu_delta, _swaps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1601_04359_amd import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("W,H,cx,cy,mask,n", [
    (2, 1, 0, 0, 3, 1), (3, 40, 2, 39, 3, 31), (40, 3, 39, 2, 1, 32), (65, 33, 12, 12, 2, 33),
    (66, 66, 63, 63, 3, 40), (70, 70, 64, 12, 3, 65), (130, 9, 126, 8, 2, 300)])
def test_partial_words_and_sectors(ctx, W, H, cx, cy, mask, n):
    print(f"[gpu] swap {W}x{H} c=({cx},{cy}) mask={mask} n={n}", flush=True)
    img = (wl.random_binary(W, H, 0.7, 5 * W + H) | wl.stripes(W, H, 16, 5)).astype(np.uint8)
    img.flat[0], img.flat[-1] = 1, 0
    ones, zeros = np.flatnonzero(img == 1), np.flatnonzero(img == 0)
    g = np.random.default_rng(W + H + n)
    sw = np.stack([g.choice(ones, n), g.choice(zeros, n)], 1).astype(np.int32)
    sw[::3] = sw[::3, ::-1]  # either order of the two phases
    if n > 4:
        sw[1], sw[3] = (0, 0), (-1, 5)  # no interchange: no change
    ok = np.array([i for i in range(n) if not (n > 4 and i in (1, 3))])
    got = _gpu_delta(ctx, img, cx, cy, sw, mask)
    assert np.array_equal(got[ok], oracle.delta_swap(img, cx, cy, sw[ok], mask))
    if n > 4:
        assert not got[1].any() and not got[3].any()


def test_scratch_batches_equal_runs(ctx):
    from paper_1601_04359_amd import _abi
    W, H, c, n = 140, 130, 100, 6000  # 102 groups of 32 candidates per batch
    print(f"[gpu] swap {W}x{H} c={c} n={n}", flush=True)
    img = wl.boolean_disks(W, H, 12.0, 0.5, 9)
    sw = _swaps(img, n, 4)
    got = _gpu_delta(ctx, img, c, c, sw[:, ::-1])
    _abi.lpf_set_delta_method(ctx.handle, _abi.LPF_SWAP_RUNS)
    try:
        for i in (0, 3200, n - 60):
            assert np.array_equal(got[i:i + 60], _gpu_delta(ctx, img, c, c, sw[i:i + 60])), i
    finally:
        _abi.lpf_set_delta_method(ctx.handle, _abi.LPF_SWAP_AUTO)


@pytest.mark.parametrize("W,H,cx,cy,mask", [(200, 40, 127, 12, 3), (300, 20, 200, 5, 2), (30, 520, 20, 255, 1)])
def test_larger_cutoffs_by_offset_rows(ctx, W, H, cx, cy, mask):
    print(f"[gpu] swap {W}x{H} c=({cx},{cy}) mask={mask}", flush=True)
    img = wl.boolean_disks(W, H, 5.0, 0.5, W)
    sw = _swaps(img, 20, 8, near=6)
    assert np.array_equal(_gpu_delta(ctx, img, cx, cy, sw, mask), oracle.delta_swap(img, cx, cy, sw, mask))
