"""Anchor sums of the interpolation decoder against the oracle: one and two
anchors per axis, lines around a wave's step (64) and its batch (256), and
around the length from which a line is cut into segments (2048 anchors,
segments of 512), with one and several lines."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1,), (8,), (9,), (17,), (8 * 64,), (8 * 64 + 1,), (8 * 256 + 1,), (8 * 2048,),
                                   (8 * 2048 + 1,), (8 * 2559 + 3,), (8 * 2560 + 1,), (8 * 70000 + 5,),
                                   (9, 8 * 2048 + 1), (40, 8 * 2700), (8 * 2049, 17), (8 * 300, 24),
                                   (8 * 2048 + 8, 9, 9), (9, 8 * 2048 + 8, 9), (9, 9, 8 * 2048 + 9), (70, 66, 520)])
def test_anchor_lines(fz, shape):
    r = np.random.default_rng(int(np.prod(shape)) % 2 ** 31)
    x = (np.cumsum(r.normal(0, 1, int(np.prod(shape)))).reshape(shape)).astype(np.float32)
    ctx = fz.Context(0)
    c = ctx.compress(torch.from_numpy(x).cuda(), 1e-3, pred=fz.PRED_INTERP)
    ref = oracle.decompress(c.cpu().numpy().tobytes()).reshape(shape)
    got = ctx.decompress(c).cpu().numpy()
    assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))
