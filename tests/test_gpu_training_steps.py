"""Whole training runs against the same steps in fp64: initial weights and
sample order from the seed, ragged last minibatches, at least four epochs (both
order buffers are used again), bias corrections by step, per-epoch losses, and
more epochs than losses are held on the device (1024).

The bounds separate fp32 rounding from a wrong step.  On the CPU, over the
cases below, the same steps in fp32 are off from fp64 by at most 2.5e-7 of a
tensor's norm and 1e-6 of a loss (a hidden unit gated the other way may add to
it: 3e-5 seen over 64 steps); a step number off by one moves W1 to W3 by 3e-3 or
more, one epoch in the order of the epoch before it by 4e-4 (its loss by
1e-4), and epochs' losses lie 5e-3 or more apart.  So 1e-4 for the weights, 1e-5
for the losses.  Over 1030 epochs fp32 is off by up to 6e-6 and the losses
around the 1024th epoch lie 8e-2 apart: 1e-4.
"""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

TENSORS = ("W1", "W2", "W3")


def splitmix(state):
    """Steele, Lea and Flood's generator: (state, value)."""
    mask = (1 << 64) - 1
    state = (state + 0x9E3779B97F4A7C15) & mask
    z = state
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & mask
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
    return state, z ^ (z >> 31)


def samples(n, seed):
    r = np.random.default_rng(seed)
    base = r.uniform(0.0, 12.0, (n, 1))
    feat = np.abs(base * r.uniform(0.2, 1.0, (1, 16)) + r.normal(0, 0.6, (n, 16))).astype(np.float32)
    bits = np.clip(feat @ r.normal(0, 0.12, (16, 3)) + 0.45 * base + 7.0 + r.normal(0, 0.2, (n, 3)), 5.0, 14.5)
    return feat, np.floor(np.exp2(bits)).astype(np.int32)


def initial(feat, seed):
    """mu and 1 / std of the features, then each layer's weights and biases
    uniform within 1 / sqrt(fan-in)."""
    w = np.zeros(oracle.NPARAM, np.float64)
    f = feat.astype(np.float64)
    o, k = oracle.OFF["mu"]
    w[o:o + k] = f.mean(0).astype(np.float32)
    o, k = oracle.OFF["rs"]
    w[o:o + k] = (1.0 / f.std(0)).astype(np.float32)
    state = seed
    for name, bias, fan in (("W1", "b1", 16), ("W2", "b2", 64), ("W3", "b3", 64)):
        o, k = oracle.OFF[name]
        for i in range(o, o + k + oracle.OFF[bias][1]):
            state, z = splitmix(state)
            w[i] = np.float32((2.0 * ((z >> 11) + 0.5) * 2.0 ** -53 - 1.0) / np.sqrt(fan))
    return w


def train(feat, costs, epochs, batch, lr, seed, grad=oracle.mlp_loss_grad, adam=oracle.adam_step):
    """Minibatch Adam in fp64: (parameters, losses per epoch)."""
    n = len(feat)
    w = initial(feat, seed)
    m, v = np.zeros_like(w), np.zeros_like(w)
    target = np.log2(1.0 + costs.astype(np.float64))
    perm, order, t, losses = list(range(n)), seed ^ 0x5DEECE66D, 0, []
    for _ in range(epochs):
        for i in range(n - 1, 0, -1):
            order, z = splitmix(order)
            j = z % (i + 1)
            perm[i], perm[j] = perm[j], perm[i]
        each = []
        for at in range(0, n, batch):
            k = perm[at:at + batch]
            loss, g = grad(w, feat[k], target[k])
            each.append(loss)
            t += 1
            adam(w, m, v, g, t, lr=float(np.float32(lr)), b1=float(np.float32(0.9)), b2=float(np.float32(0.999)),
                 eps=float(np.float32(1e-8)))
        losses.append(float(np.mean(each)))
    return w, np.array(losses)


CASES = [(100, 32, 5, 1e-3), (77, 16, 6, 2e-3), (33, 33, 7, 1e-3), (1000, 256, 4, 1e-3), (5, 1, 4, 1e-3)]


@pytest.mark.parametrize("n,batch,epochs,lr", CASES)
def test_steps_and_losses(fz, n, batch, epochs, lr):
    feat, costs = samples(n, n)
    ctx = fz.Context(0)
    loss = ctx.selector_train(torch.from_numpy(feat).cuda(), torch.from_numpy(costs).cuda(), epochs=epochs, batch=batch,
                              lr=lr, seed=n + 1)
    w, ref = train(feat, costs, epochs, batch, lr, n + 1)
    assert np.all(np.abs(loss - ref) <= 1e-5 * ref), np.abs(loss / ref - 1).max()
    got = np.asarray(ctx.selector_get(), np.float64)
    for name in TENSORS:
        o, k = oracle.OFF[name]
        e = np.linalg.norm(got[o:o + k] - w[o:o + k]) / np.linalg.norm(w[o:o + k])
        assert e <= 1e-4, (name, e)


@pytest.mark.parametrize("epochs", [1024, 1025, 1030])
def test_losses_of_many_epochs(fz, epochs):
    # (a small step keeps the run of 2 steps an epoch close to fp64)
    feat, costs = samples(20, 3)
    ctx = fz.Context(0)
    loss = ctx.selector_train(torch.from_numpy(feat).cuda(), torch.from_numpy(costs).cuda(), epochs=epochs, batch=16,
                              lr=3e-5, seed=9)
    ref = train(feat, costs, epochs, 16, 3e-5, 9)[1]
    assert np.all(np.abs(loss - ref) <= 1e-4 * ref), np.abs(loss / ref - 1).max()
