"""The wave-per-block decoder on codes that hardly fall into step (codewords
nearly all 8 bits long, in full blocks and in blocks of few values), where it
leaves the rounds for the walk from every possible start, and on codes in
between.  Reconstructions equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

SHAPES = [(1,), (7,), (512,), (4099,), (1, 700), (3, 700), (17, 300), (64, 96), (1, 33, 40), (9, 41, 40), (24, 24, 24)]


@pytest.fixture(scope="module")
def ctx(fz):
    return fz.Context(0)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("levels", [128, 256, 300])
@pytest.mark.parametrize("pred", [0, 2])
def test_equally_long_codewords(fz, ctx, shape, levels, pred):
    # residuals (nearly) uniform over `levels` values: steps along x for the
    # first-order predictor, the values themselves for the other two
    r = np.random.default_rng(levels + len(shape))
    x = r.integers(0, levels, shape) - levels // 2
    if pred == 0:
        for axis in range(len(shape)):
            x = np.cumsum(x, axis=axis)
    x = x.astype(np.float32)
    c = ctx.compress(torch.from_numpy(x).cuda(), 0.5, 0, pred=pred)
    ref = np.asarray(oracle.decompress(c.cpu().numpy().tobytes()), np.float32).reshape(shape)
    assert np.array_equal(ctx.decompress(c).cpu().numpy().view(np.uint32), ref.view(np.uint32))
