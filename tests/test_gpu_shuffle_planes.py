"""The bit-shuffle codec where its kernels take other paths: blocks whose
symbols fill 1 to 10 planes (steps of the decoder at 4 and 8), with and
without outliers, several kinds in one field, block counts around the copy's
groups, in 1D, 2D and 3D.  Containers and reconstructions equal the
oracle's."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

SHAPES = [(512,), (513,), (512 * 15 + 3,), (512 * 64,), (512 * 65 + 511,), (16, 32), (50, 97), (8, 8, 8), (17, 24, 33),
          (40, 40, 40)]


def _field(shape, top, seed):
    """Integers whose residuals along the last axis stay below `top` a block
    (0: every block its own)."""
    r = np.random.default_rng(seed)
    n = int(np.prod(shape))
    tops = np.full(n, float(top)) if top else 2.0 ** r.integers(0, 10, (n + 511) // 512).repeat(512)[:n]
    d = np.rint(r.uniform(-1, 1, n) * tops)
    d = np.where(r.random(n) < 0.7, 0, d).reshape(shape)
    for axis in range(len(shape)):
        # the inverse of the block-wise differences, block by block
        ext = {1: [512], 2: [16, 32], 3: [8, 8, 8]}[len(shape)][axis]
        for i0 in range(0, shape[axis], ext):
            sl = [slice(None)] * len(shape)
            sl[axis] = slice(i0, i0 + ext)
            d[tuple(sl)] = np.cumsum(d[tuple(sl)], axis=axis)
    return (d * 2e-3).astype(np.float32)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("top", [0, 1, 7, 8, 100, 127, 129, 500, 700])
def test_planes(fz, shape, top):
    ctx = fz.Context(0)
    x = _field(shape, top, seed=sum(shape) + top)
    c = ctx.compress(torch.from_numpy(x).cuda(), 1e-3, fz.EB_ABS, codec="shuffle")
    b = c.cpu().numpy().tobytes()
    assert b == oracle.speed_compress(x, 1e-3, 0)
    ref = np.asarray(oracle.decompress(b), np.float32).reshape(shape)
    assert np.array_equal(ctx.decompress(c).cpu().numpy().view(np.uint32), ref.view(np.uint32))
