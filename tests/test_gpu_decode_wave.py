"""The wave-per-block decoder against the oracle, at the sizes where it
can go wrong: single values, blocks cut along each axis, fields with only
edge blocks, the largest field it takes whole and the smallest whose
interior goes to the lane decoder, every predictor; codes that fall into
step late (all codewords equally long, so every lane waits for the one
before it) and blocks of outliers."""
import numpy as np
import pytest
import torch

import oracle
from inputs import fields

pytestmark = pytest.mark.gpu

LIMIT = 16384  # blocks


@pytest.fixture(scope="module")
def ctx(fz):
    return fz.Context(0)


def _check(fz, ctx, x, eb, pred, mode=1):
    d = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    c = ctx.compress(d, eb, mode, pred=pred)
    ref = oracle.decompress(c.cpu().numpy().tobytes())
    got = ctx.decompress(c).cpu().numpy()
    assert np.array_equal(got.view(np.uint32), ref.reshape(got.shape).view(np.uint32))
    return fz.header_fields(c[:128].cpu().numpy().tobytes())


@pytest.mark.parametrize("pred", [0, 1, 2, 4, 5, 6])
@pytest.mark.parametrize("shape", [(1,), (511,), (513,), (5000,), (1, 1), (15, 31), (16, 33), (33, 95), (1, 1, 1),
                                   (7, 7, 7), (9, 16, 23), (8, 40, 64), (17, 8, 8)])
def test_shapes_and_predictors(fz, ctx, shape, pred):
    x = fields.random_small(shape, seed=5, kind="smooth")
    for eb in (1e-2, 1e-4):
        _check(fz, ctx, x, eb, pred)


@pytest.mark.parametrize("blocks,extra", [(LIMIT, 0), (LIMIT - 1, 1), (LIMIT, 1), (LIMIT, 511), (LIMIT + 3, 0)])
def test_limit(fz, ctx, blocks, extra):
    x = fields.sorted_positions(512 * blocks + extra, seed=blocks + extra)
    _check(fz, ctx, x, 1e-5, 0)


@pytest.mark.parametrize("pred", [0, 5, 6])
def test_edges_of_a_large_field(fz, ctx, pred):
    # 41 x 21 x 21 blocks, every axis cut
    x = fields.grf((321, 165, 163), alpha=3.0, seed=9)
    _check(fz, ctx, x, 1e-3, pred)


@pytest.mark.parametrize("levels", [2, 4, 64, 512, 1000])
def test_late_synchronisation(fz, ctx, levels):
    # 1D, absolute bound 0.5: the residuals are the steps, uniform over
    # `levels` values, so all codewords have nearly the same length
    r = np.random.default_rng(levels)
    x = np.cumsum(r.integers(0, levels, 20_000) - levels // 2).astype(np.float32)
    _check(fz, ctx, x, 0.5, 0, mode=0)


def test_blocks_of_outliers(fz, ctx):
    r = np.random.default_rng(1)
    x = r.uniform(-1, 1, (24, 24, 24)).astype(np.float32)
    x[:8, :8, :8] *= 4000.0
    x[8:, 8:16] = 0.25
    h = _check(fz, ctx, x, 0.5, 0, mode=0)
    assert h["n_outliers"] > 400


def test_damaged_chunk_table(fz, ctx):
    x = torch.from_numpy(fields.sinusoid_field((24, 24, 24), seed=2)).cuda()
    c = ctx.compress(x, 1e-3)
    for k, v in ((0, 65535), (3, 0), (5, 6145), (26, 1)):
        bad = c.clone()
        at = 128 + 512 + 2 * k
        bad[at] = v & 255
        bad[at + 1] = v >> 8
        with pytest.raises(fz.FZError) as e:
            ctx.decompress(bad)
        assert e.value.code == -5
