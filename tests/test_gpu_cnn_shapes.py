"""The network's layered kernels at the edges of their strips (16 pixels wide; 8 rows high, 16 for
the weights' gradients) against the float64 oracle on bf16-rounded values.

Tolerance.  Scores: as in test_gpu_cnn.py.  Gradients: both sides round the same values to bf16 at
the same places; where a sum falls next to a rounding boundary they differ by one unit, 2^-8 of one
of the 2 n sampled pixels' terms, and the terms of a gradient have either sign, so one such value
moves it by 2^-8 / sqrt(2 n) of its scale; four of them are allowed: 2^-6 / sqrt(2 n).  A pixel left
out or counted twice moves it by 1 / sqrt(2 n).  Scale: the group's RMS or the whole gradient's,
the larger (a group can cancel)."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl
from oracle import cnn
from test_gpu_cnn import _bits, _close, _groups, _net, _params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,batch,n", [(1, 1, 2, 4), (15, 7, 3, 40), (16, 8, 1, 64), (17, 9, 2, 255),
                                         (33, 16, 3, 256), (48, 17, 2, 257), (70, 35, 4, 600)])
def test_layers_at_strip_edges(W, H, batch, n):
    import torch
    from paper_1601_04359_amd import Context, cnn_samples
    print(f"[gpu] cnn {W}x{H} batch {batch} samples {n}", flush=True)
    g = np.random.default_rng(W * 100 + H)
    prm = _params(W + H)
    imgs = [wl.random_binary(W, H, 0.4, 60 + W + i) for i in range(batch)]
    idx = g.integers(0, batch, n)
    a, b = g.integers(0, W * H, n), g.integers(0, W * H, n)
    y = g.normal(size=n).astype(np.float32)
    with Context(0) as ctx:
        net, bits = _net(ctx, W, H, batch, n, prm), _bits(ctx, imgs)
        S = net.forward(bits, batch).cpu().numpy()
        for i, im in enumerate(imgs):
            _close(S[i], cnn.forward(prm, im)["S"])
        grad, loss = net.grad(bits, batch, cnn_samples(idx, a, b, y, "cuda"))
        ref_loss, ref = cnn.loss_and_grad(prm, imgs, np.stack([idx, a, b, y], 1))
        assert abs(float(loss.cpu()[0]) - ref_loss) <= 2.0 ** -6 / np.sqrt(2 * n) * ref_loss
        got = grad.cpu().numpy().astype(np.float64)
        whole = np.sqrt(np.mean(ref ** 2))
        for k, off, size in _groups():
            gk, rk = got[off:off + size], ref[off:off + size]
            scale = max(np.sqrt(np.mean(rk ** 2)), whole)
            assert np.max(np.abs(gk - rk)) <= 2.0 ** -6 / np.sqrt(2 * n) * scale, k
        # after a step the layers use the new parameters' bf16 weights
        net.adam(grad, 1e-3)
        fresh = _net(ctx, W, H, batch, n, net.params().cpu().numpy())
        assert torch.equal(net.forward(bits, batch), fresh.forward(bits, batch))
        net.close()
        fresh.close()
