"""Batches whose fields lie on both sides of the sizes at which a batch's
decode changes from a wave to a lane per block (earlier in 3D than for a
single field): every field equals its single call's."""
import numpy as np
import pytest
import torch

from inputs import fields

pytestmark = pytest.mark.gpu

SHAPES = [(144, 144, 144), (152, 152, 152), (149, 150, 151), (192, 192, 192), (190, 191, 189), (1800, 3600), (2048, 3072),
          (512 * 12288,), (1, 40000), (12, 300, 300)]


@pytest.mark.parametrize("pred,eb", [(0, 1e-2), (2, 2e-4)])
def test_batch_equals_single_calls(fz, pred, eb):
    ctx = fz.Context(0)
    xs = [torch.from_numpy(fields.random_small(s, seed=k, kind="smooth")).cuda() for k, s in enumerate(SHAPES)]
    for k, x in enumerate(xs):
        g = torch.Generator(device="cuda")
        g.manual_seed(k)
        x.add_(torch.randn(x.shape, generator=g, device="cuda"), alpha=0.02 * float(x.max() - x.min()))
    packed, offs = ctx.compress_batch(xs, [eb] * len(xs), preds=[pred] * len(xs))
    outs = [torch.empty_like(x) for x in xs]
    for _ in range(2):  # captured, then replayed
        ctx.decompress_batch(packed, offs, outs)
        for x, y in zip(xs, outs):
            c = ctx.compress(x, eb, pred=pred)
            assert torch.equal(y.view(torch.int32), ctx.decompress(c).view(torch.int32))
            y.zero_()
