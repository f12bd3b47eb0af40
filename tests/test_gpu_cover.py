"""lpf_full's cover kernel at the edges of its shapes: every lane width, partial words and bands,
tiles down and across, split groups, against the oracle (all counts, exact)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as wl

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


# W = 32 R - (0, 1 or 31): one lane of R words per row; the image height leaves a partial band
@pytest.mark.parametrize("R", list(range(1, 17)))
def test_lane_widths(ctx, R):
    import torch
    W, H, cx, cy = 32 * R - (0, 1, 31)[R % 3], 65 + R, min(20, 32 * R - 32), 18
    print(f"[gpu] cover {W}x{H} cutoff ({cx}, {cy})", flush=True)
    img = wl.boolean_disks(W, H, 5.0, 0.5, 40 + R)
    bits = ctx.pack(torch.from_numpy(img).cuda())
    ref = oracle.lpf(img, cx, cy, 3)
    got = ctx.full(bits, W, H, cx, cy)
    enh = ctx.full_enhanced(bits, W, H, cx, cy)
    sample = wl.sample_positions(W, H, W * H // 3, R)
    smp = ctx.full_sampled(bits, W, H, cx, cy, ctx.pack(torch.from_numpy(sample).cuda()))
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().astype(np.uint32), ref)
    assert np.array_equal(enh.cpu().numpy().astype(np.uint32), ref)
    assert np.array_equal(smp.cpu().numpy().astype(np.uint32), oracle.lpf_sampled(img, cx, cy, sample, 3))


@pytest.mark.parametrize("W,H,cx,cy,mask,layout", [
    (900, 300, 20, 120, 3, 1),   # tiles across and down, groups split over workgroups, GRID
    (1030, 33, 40, 32, 1, 0),    # a row of three tiles, the last a single word
    (600, 1100, 12, 9, 2, 0),    # many row tiles
    (17, 300, 16, 150, 3, 0),    # rows narrower than a word, wrapped several times
    (31, 31, 30, 30, 3, 1),      # whole domain
    (2, 2, 1, 1, 3, 0),
])
def test_tiles_and_layouts(ctx, W, H, cx, cy, mask, layout):
    import torch
    print(f"[gpu] cover {W}x{H} cutoff ({cx}, {cy}) mask {mask} layout {layout}", flush=True)
    img = wl.random_binary(W, H, 0.8, W + H) | wl.checkerboard(W, H, 3)
    bits = ctx.pack(torch.from_numpy(img.astype(np.uint8)).cuda())
    out = ctx.full(bits, W, H, cx, cy, mask, layout)
    out.fill_(-1)  # written in full
    ctx.full(bits, W, H, cx, cy, mask, layout, out=out)
    torch.cuda.synchronize()
    ref = oracle.lpf(img.astype(np.uint8), cx, cy, mask, layout=layout)
    assert np.array_equal(out.cpu().numpy().astype(np.uint32), ref)


def test_dirty_padding_bits_are_ignored(ctx):
    # bits past W in the last word of a row are not part of the image
    import torch
    W, H = 75, 70
    img = wl.boolean_disks(W, H, 5.0, 0.5, 2)
    bits = ctx.pack(torch.from_numpy(img).cuda())
    dirty = bits.clone()
    dirty[:, 1] |= -(1 << 11)  # bits 75.. of each row
    a = ctx.full(bits, W, H, 30, 25)
    b = ctx.full(dirty, W, H, 30, 25)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
    assert np.array_equal(a.cpu().numpy().astype(np.uint32), oracle.lpf(img, 30, 25, 3))
