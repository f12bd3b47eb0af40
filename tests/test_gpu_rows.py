"""lpf_full, _enhanced, _sampled and lpf_batch on images of a few rows longer than 1024 pixels (64
lanes per row, tiles of one row and a few), against the oracle.  Whole numbers, no tolerance."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

SIZES = [(1040, 1, 300, 0), (2048, 1, 1000, 0), (2048, 2, 400, 1), (2049, 3, 260, 2), (20000, 1, 500, 0)]


def _image(W, H):
    img = np.ones((H, W), np.uint8)
    img[:, W // 5] = 0
    img[H // 2, W // 2: W // 2 + 200] = wl.random_binary(200, 1, 0.8, W)[0]
    return img


def test_few_long_rows():
    import torch
    from paper_1601_04359_amd import Context
    with Context(0) as ctx:
        items, refs = [], []
        for W, H, cx, cy in SIZES:
            print(f"[gpu] rows {W}x{H} cutoff ({cx}, {cy})", flush=True)
            img = _image(W, H)
            bits = ctx.pack(torch.from_numpy(img).cuda())
            ref = oracle.lpf(img, cx, cy, 3)
            sample = wl.sample_positions(W, H, W * H // 3, 1)
            for got, want in ((ctx.full(bits, W, H, cx, cy), ref),
                              (ctx.full_enhanced(bits, W, H, cx, cy), ref),
                              (ctx.full_sampled(bits, W, H, cx, cy, ctx.pack(torch.from_numpy(sample).cuda())),
                               oracle.lpf_sampled(img, cx, cy, sample, 3))):
                assert np.array_equal(got.cpu().numpy().astype(np.uint32), want)
            items.append((bits, W, H, cx, cy))
            refs.append(ref)
        print("[gpu] rows batch", flush=True)
        counts, offs, _, _ = ctx.batch(items, 3, 0)
        c = counts.cpu().numpy().astype(np.uint32)
        for o, ref in zip(offs, refs):
            assert np.array_equal(c[o:o + ref.size], ref.reshape(-1))
