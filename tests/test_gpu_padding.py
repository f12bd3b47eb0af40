"""Bits past the width in the last word of a packed row are no part of the image: every call that
reads packed rows gives the same results whatever they are, for rows narrower than a word too."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


def _dirty(bits, W):
    d = bits.clone()
    if W % 64:
        d[..., -1] |= -(1 << (W % 64))
    return d


@pytest.mark.parametrize("W,H", [(1, 70), (5, 40), (20, 34), (31, 64), (33, 20), (75, 70), (128, 20)])
def test_padding_is_ignored(W, H):
    import torch
    from paper_1601_04359_amd import Context
    print(f"[gpu] padding {W}x{H}", flush=True)
    img = (wl.random_binary(W, H, 0.8, W) | wl.stripes(W, H, 16, 5)).astype(np.uint8)
    img.flat[0], img.flat[-1] = 1, 0
    cx, cy = min(W - 1, 12), 10
    ones, zeros = np.flatnonzero(img == 1), np.flatnonzero(img == 0)
    g = np.random.default_rng(W)
    sw = np.stack([g.choice(ones, 70), g.choice(zeros, 70)], 1).astype(np.int32)
    sample = wl.sample_positions(W, H, W * H // 2, 1)
    with Context(0) as ctx:
        bits = _dirty(ctx.pack(torch.from_numpy(img).cuda()), W)
        mask = _dirty(ctx.pack(torch.from_numpy(sample).cuda()), W)
        swaps = torch.from_numpy(sw).cuda()

        def same(got, ref):
            assert np.array_equal(got.cpu().numpy().astype(np.int64), ref.astype(np.int64))
        same(ctx.full(bits, W, H, cx, cy), oracle.lpf(img, cx, cy, 3))
        same(ctx.full_sampled(bits, W, H, cx, cy, mask), oracle.lpf_sampled(img, cx, cy, sample, 3))
        same(ctx.s2(bits, W, H, cx, cy), oracle.s2(img, cx, cy, 3))
        same(ctx.delta_swap(bits, W, H, cx, cy, swaps), oracle.delta_swap(img, cx, cy, sw, 3))
        same(ctx.full3d(bits.view(H, -1), W, H // 2, 2, cx, 4, 1),
             oracle.lpf3(img[:H // 2 * 2].reshape(2, H // 2, W), cx, 4, 1, 3))
