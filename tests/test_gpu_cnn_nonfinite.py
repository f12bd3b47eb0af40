"""A value that is not finite stays in its own channel of the network's weight gradients.

Channel 5 of layer 1 overflows at the interfaces, rows 0 to 8 of each image, and the samples lie
more than the network's reach (3 pixels) away, so that the loss and the score gradient are finite and
only the activations of the upper rows are not: there the gradients of layer 2's weights are 0 * inf for
input channel 5 and 0 * finite for the others.  Weights into layers 2 and 3 are not negative, so that
no inf - inf appears on the way and the oracle's ReLU and the kernels' see the same values.

Tolerance.  The sampled rows are one phase, so their activations are alike: where one falls next to a
rounding boundary, both sides may differ by one unit, 2^-8, at every sample at once, which moves a
gradient by 2^-8 of its largest entry; four such values are allowed, 2^-6."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import cnn
from test_gpu_cnn import _bits, _net, _params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,n", [(33, 40, 200), (64, 48, 500)])
def test_other_channels_stay_finite(W, H, n):
    from paper_1601_04359_amd import Context, cnn_samples
    print(f"[gpu] cnn non-finite {W}x{H}", flush=True)
    p = cnn.unpack(_params(9).astype(np.float64))
    p["W1"][:, 5, 1] = 3e38  # three taps of a full interface row overflow
    p["W2"], p["W3"] = np.abs(p["W2"]), np.abs(p["W3"])
    prm = cnn.pack(p)
    img = np.zeros((H, W), np.uint8)
    img[0:8:2] = 1  # full rows: interfaces in rows H - 1 and 0 to 7
    g = np.random.default_rng(W)
    lo, hi = 13 * W, (H - 6) * W
    a, b = g.integers(lo, hi, n), g.integers(lo, hi, n)
    idx, y = np.zeros(n, int), (50 * g.normal(size=n)).astype(np.float32)
    with np.errstate(all="ignore"):
        f = cnn.forward(prm, img)
        assert np.isinf(f["A1"][..., 5]).any() and np.isfinite(np.delete(f["A1"], 5, 2)).all()
        ref_loss, ref = cnn.loss_and_grad(prm, [img], np.stack([idx, a, b, y], 1))
    with Context(0) as ctx:
        net = _net(ctx, W, H, 1, n, prm)
        grad, loss = net.grad(_bits(ctx, [img]), 1, cnn_samples(idx, a, b, y, "cuda"))
        got, loss = grad.cpu().numpy().astype(np.float64), float(loss.cpu()[0])
        net.close()
    assert np.isfinite(loss) and abs(loss - ref_loss) <= 2.0 ** -6 * ref_loss
    got, ref = cnn.unpack(got), cnn.unpack(ref)
    finite = np.isfinite(ref["W2"])
    assert finite.any() and not finite[..., 5].any() and finite[..., np.arange(16) != 5].all()
    for k in ("W1", "b1", "W2", "b2", "b3", "b4"):
        ok = np.isfinite(ref[k])
        assert np.array_equal(np.isfinite(got[k]), ok), k
        scale = max(np.max(np.abs(ref[k][ok])), np.max(np.abs(ref["W2"][finite])))
        assert np.max(np.abs(got[k][ok] - ref[k][ok])) <= 2.0 ** -6 * scale, k
