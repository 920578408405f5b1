"""Gradient and loss of the selector at batch sizes around the edges of the
training kernel's split: one sample, a tile of 16 and its neighbours, the
512 tiles that get a workgroup each and one sample more, and several tiles
per workgroup with a ragged last one.

Against the oracle's fp64 backpropagation.  A gradient is a sum over the
batch of products of 64-term dot products in fp32: relative error below
(64 + 64 + 16) roundings of 6e-8, 1e-5; a hidden unit within rounding of
zero may be gated the other way, which moves one of the batch's terms, so
the bound is 1e-4 for the gradient (1e-5 for the loss)."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 1023, 8192, 8193, 20011])
def test_gradient_at_split_edges(fz, n):
    r = np.random.default_rng(n)
    ctx = fz.Context(0)
    w = r.normal(0, 0.25, oracle.NPARAM).astype(np.float32)
    o, k = oracle.OFF["mu"]
    w[o:o + k] = r.uniform(0, 3, k)
    o, k = oracle.OFF["rs"]
    w[o:o + k] = r.uniform(0.5, 1.5, k)
    ctx.selector_set(w)
    feat = r.uniform(0, 6, (n, 16)).astype(np.float32)
    tgt = r.uniform(0, 12, (n, 3)).astype(np.float32)
    g, loss = ctx.selector_grad(torch.from_numpy(feat).cuda(), torch.from_numpy(tgt).cuda())
    lo, go = oracle.mlp_loss_grad(w.astype(np.float64), feat, tgt.astype(np.float64))
    assert abs(loss - lo) <= 1e-5 * lo
    assert np.all(g[:oracle.OFF["W1"][0]] == 0)
    for name in ("W1", "b1", "W2", "b2", "W3", "b3"):
        o, k = oracle.OFF[name]
        e = np.linalg.norm(g[o:o + k] - go[o:o + k]) / max(np.linalg.norm(go[o:o + k]), 1e-30)
        assert e <= 1e-4, (name, e)
