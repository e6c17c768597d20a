"""The training gradient where its tiles of 32 samples, groups of four tiles and
rounds of a block leave a remainder, against the FP64 oracle.

A gradient is a sum over the batch of products of FP32 sums of up to 64 terms
(two layers forward, two back): some 200 roundings of 6e-8 deep, 1.2e-5 of the
terms' size, and the terms cancel to an eighth of it at most for these inputs,
so 1e-4 of a layer's norm bounds it."""
import numpy as np
import pytest

import pyoracle as O

pytestmark = pytest.mark.gpu

T = pytest.importorskip("paper_2011_00459_amd.terrain")
D = pytest.importorskip("paper_2011_00459_amd.devmem")
LN = pytest.importorskip("paper_2011_00459_amd.learn")

LAYERS = (("W1", (64, 12)), ("b1", (64,)), ("W2", (64, 64)), ("b2", (64,)), ("W3", (3, 64)), ("b3", (3,)))


# one, two and four rounds a block: up to 32,768, up to 98,304 and more samples
@pytest.mark.parametrize("n", [1, 31, 32, 33, 127, 128, 129, 1000, 32768, 32769, 98305])
def test_gradient_matches_oracle(n):
    rng = np.random.default_rng(n)
    feat = rng.normal(size=(n, 12)).astype(np.float32)
    label = (0.5 + rng.normal(size=(n, 3))).astype(np.float32)
    flat = LN.flatten(LN.init_weights(3, rng.uniform(0.3, 1.0, 12).astype(np.float32)))
    ns = T.mlp_grad_scratch_floats(n)
    W, F, L = (D.DeviceArray.from_host(a, np.float32) for a in (flat, feat, label))
    G, loss, S = D.DeviceArray((T.MLP_TRAINABLE,), np.float32), D.DeviceArray((1,), np.float32), D.DeviceArray((ns,), np.float32)
    T.mlp_loss_grad(W.ptr, F.ptr, L.ptr, n, G.ptr, loss.ptr, S.ptr, ns)
    grad = G.get()
    loss_ref, ref = O.mlp_loss_grad(LN.unflatten(flat), feat.astype(np.float64), label.astype(np.float64))
    assert loss.get()[0] == pytest.approx(loss_ref, rel=1e-4)
    o = 0
    for k, shp in LAYERS:
        g = grad[o:o + int(np.prod(shp))].reshape(shp)
        o += g.size
        assert np.linalg.norm(g - ref[k]) <= 1e-4 * np.linalg.norm(ref[k]), k
