"""Containers against the oracle where the quantiser takes its other paths:
tiles of four 8^3 blocks that do and do not lie side by side (rows of 1 to 9
blocks, ragged ends, axes of one value), and values whose lossless-patch test
is close (just inside and outside the bound, near the largest grid value, no
finite value, bounds below the smallest normal float), in blocks and in their
neighbours' halos."""
import numpy as np
import pytest
import torch

import oracle
from inputs import fields

pytestmark = pytest.mark.gpu

SHAPES = [(9, 9, 8), (17, 8, 25), (8, 24, 32), (16, 17, 33), (10, 11, 64), (1, 1, 300), (25, 1, 65), (1, 40, 72),
          (33, 34, 63)]


def _edge_values(shape, eb, seed):
    """A smooth field with values at the edges of the patch test strewn in."""
    x = (fields.random_small(shape, seed=seed, kind="smooth") * np.float64(300 * eb)).astype(np.float32)
    r = np.random.default_rng(seed)
    f = x.reshape(-1)
    at = r.choice(f.size, size=max(1, f.size // 40), replace=False)
    big = np.float64(2 * eb) * 2.0**24
    cand = np.array([big, -big, big * (1 - 2.0**-18), big * (1 + 2.0**-18), big / 2 + eb, 7 * eb, -9 * eb, 1e30, -0.0])
    f[at] = cand[r.integers(0, cand.size, at.size)].astype(np.float32)
    return x


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("pred", [oracle.P0, oracle.P_INTERP, oracle.P_GLOBAL])
def test_tiles_and_patch_edges(fz, shape, pred):
    ctx = fz.Context(0)
    for eb in (1e-3, 3e-39):
        x = _edge_values(shape, eb, seed=sum(shape))
        c = ctx.compress(torch.from_numpy(x).cuda(), eb, mode=fz.EB_ABS, pred=pred).cpu().numpy().tobytes()
        assert c == oracle.compress(x, eb, 0, pred=pred)


@pytest.mark.parametrize("shape", [(1025,), (33, 47), (9, 10, 35)])
def test_not_finite(fz, shape):
    ctx = fz.Context(0)
    x = fields.random_small(shape, seed=1, kind="smooth")
    x.reshape(-1)[-1] = np.nan
    with pytest.raises(fz.FZError) as e:
        ctx.compress(torch.from_numpy(x).cuda(), 1e-3, mode=fz.EB_ABS)
    assert e.value.code == -3
