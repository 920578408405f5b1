"""Gradient of a batch that does not fill a tile of 16 samples, with biases
whose activations alone overflow fp32 while every sample's own stay small:
the slots past the batch add nothing.  Against the oracle's fp64
backpropagation, to the same 1e-4 as at ordinary parameters (about 144
roundings of 6e-8, 1e-5, and one hidden unit gated the other way)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 33])
def test_slots_past_the_batch(fz, n):
    r = np.random.default_rng(n)
    w = np.zeros(oracle.NPARAM, np.float32)
    for name in ("W1", "b1", "W2", "b2", "W3", "b3"):
        o, k = oracle.OFF[name]
        w[o:o + k] = r.normal(0, 0.25, k)
    o, k = oracle.OFF["rs"]
    w[o:o + k] = 1.0
    # unit 0 of the first layer: 1e20 from its bias, 0 for every sample
    w[oracle.OFF["b1"][0]] = 1e20
    w[oracle.OFF["W1"][0]:oracle.OFF["W1"][0] + 16] = 0.0
    w[oracle.OFF["W1"][0]] = -1e20
    w[oracle.OFF["W2"][0]] = 1e20  # unit 0 of the second layer: 1e40 in a slot past the batch
    feat = r.uniform(0, 3, (n, 16)).astype(np.float32)
    feat[:, 0] = 1.0
    tgt = r.uniform(0, 12, (n, 3)).astype(np.float32)
    ctx = fz.Context(0)
    ctx.selector_set(w)
    g, loss = ctx.selector_grad(torch.from_numpy(feat).cuda(), torch.from_numpy(tgt).cuda())
    lo, go = oracle.mlp_loss_grad(w.astype(np.float64), feat, tgt.astype(np.float64))
    assert np.all(np.isfinite(go)) and np.all(np.isfinite(g))
    assert abs(loss - lo) <= 1e-5 * lo
    for name in ("W1", "b1", "W2", "b2", "W3", "b3"):
        o, k = oracle.OFF[name]
        e = np.linalg.norm(g[o:o + k] - go[o:o + k]) / max(np.linalg.norm(go[o:o + k]), 1e-30)
        assert e <= 1e-4, (name, e)
