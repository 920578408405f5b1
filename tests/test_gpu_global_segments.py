"""Global first-order Lorenzo decode at the edges of its inverse's paths: y in
segments of 8 rows (one segment, ragged last ones, more than the segment scan
keeps in flight, rows of one wave to sixteen, ragged and unaligned), z walked
inside the segments or in a pass before them, rows too long for them, and
fields just under and over the smallest.  Reconstructions equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from inputs import fields

pytestmark = pytest.mark.gpu

SHAPES = [
    (1, 7), (8, 3), (9, 256), (17, 257), (137, 1), (300, 5), (16, 4093), (24, 4096), (11, 4097), (520, 1025),
    (3, 2048, 2050), (4, 1033, 4095), (2, 16384, 260),  # z walked
    (33, 64, 62), (32, 64, 64), (41, 61, 67), (4, 9, 4096), (150, 8, 131), (70, 1, 2048),  # z first
    (3, 200, 4100), (20, 30, 40),  # a pass per axis
]


@pytest.mark.parametrize("shape", SHAPES)
def test_segments(fz, shape):
    ctx = fz.Context(0)
    x = fields.random_small(shape, seed=sum(shape), kind="smooth")
    x.reshape(-1)[:: max(7, x.size // 50)] *= 40.0  # outliers: large sums on every axis
    c = ctx.compress(torch.from_numpy(x).cuda(), 1e-3, pred=fz.PRED_GLOBAL)
    y = ctx.decompress(c).cpu().numpy()
    ref = oracle.decompress(c.cpu().numpy().tobytes())
    assert np.array_equal(y.view(np.uint32), np.asarray(ref, np.float32).reshape(shape).view(np.uint32))
