"""Every Huffman decode path above and below the sizes at which the decoder
changes from a wave to a lane per block: interiors in lanes with scattered
edges, edges that are the last blocks, rows that do and do not allow 16-byte
stores, fields without an interior, blocks of few values, streams just long
enough for the lanes, and outputs that are not 16-byte aligned.
Reconstructions equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from inputs import fields

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fz):
    return fz.Context(0)


def _rough(shape, seed):
    """A smooth field with noise of about 100 steps of 1e-3 of its range."""
    r = np.random.default_rng(seed)
    x = np.zeros(shape, np.float64)
    for axis, n in enumerate(shape):
        view = [1] * len(shape)
        view[axis] = n
        x += np.sin(np.arange(n) * (7.0 / n) + axis).reshape(view)
    return (x + r.normal(0, 0.05, shape)).astype(np.float32)


def _check(ctx, x, eb, pred, at=0):
    c = ctx.compress(torch.from_numpy(x).cuda(), eb, 1, pred=pred)
    ref = np.asarray(oracle.decompress(c.cpu().numpy().tobytes()), np.float32).reshape(x.shape)
    buf = torch.full((x.size + at,), -7.0, device="cuda")
    got = ctx.decompress(c, out=buf[at:].view(x.shape)).cpu().numpy()
    assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))
    assert at == 0 or bool((buf[:at] == -7.0).all())


@pytest.mark.parametrize("pred", [0, 1, 2, 4, 5, 6])
@pytest.mark.parametrize("shape", [(2900, 3001), (2900, 3004), (2896, 3008)])
def test_2d_lanes(fz, ctx, shape, pred):
    _check(ctx, _rough(shape, 1), 1e-3, pred)


@pytest.mark.parametrize("pred", [0, 1, 2, 4, 5, 6])
@pytest.mark.parametrize("shape", [(321, 165, 163), (321, 165, 164), (212, 208, 208), (34, 256, 520)])
def test_3d_lanes(fz, ctx, shape, pred):
    _check(ctx, _rough(shape, 2), 1e-3, pred)


@pytest.mark.parametrize("pred", [0, 1, 2, 4, 5])
@pytest.mark.parametrize("n", [512 * 16385, 512 * 16400 + 77, 512 * 9000, 512 * 9000 + 1])
def test_1d_lanes(fz, ctx, n, pred):
    _check(ctx, _rough((n,), 3), 1e-3, pred)


# no interior, or edges of few values: 32 to 480 a block, more and fewer
# blocks than the wave takes
THIN = [(4096, 3, 260), (1, 1000, 1000), (4, 1000, 1000), (1000, 1000, 4), (9, 800, 800), (12, 400, 408),
        (1, 400000), (1, 40000), (3, 500000), (15, 300000), (17, 200000), (300000, 5), (70000, 33), (7, 7, 40000)]


@pytest.mark.parametrize("pred", [0, 2, 4, 6])
@pytest.mark.parametrize("shape", THIN)
def test_thin(fz, ctx, shape, pred):
    _check(ctx, _rough(shape, 4), 1e-3, pred)


@pytest.mark.parametrize("pred", [0, 1, 2, 4, 5, 6])
@pytest.mark.parametrize("shape", [(9_000_000,), (2896, 3008), (208, 216, 208), (512, 64, 520), (40, 48, 56)])
def test_unaligned_output(fz, ctx, shape, pred):
    _check(ctx, _rough(shape, 5), 1e-3, pred, at=1)
