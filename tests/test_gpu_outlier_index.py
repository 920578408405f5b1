"""Decoding of outlier lists at the edges of the index kernel's groups of 4
entries, waves of 64 groups, workgroups and unrolled steps, with outliers
dense enough that a row holds several; reconstructions equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 3, 4, 5, 255, 256, 257, 1023, 1025, 4095, 4097, 40961])
@pytest.mark.parametrize("every", [1, 3, 97])
def test_outlier_lists(fz, count, every):
    ctx = fz.Context(0)
    n = max(512, count * every + 7)
    r = np.random.default_rng(count * 100 + every)
    steps = r.integers(-3, 4, n).astype(np.float64)
    at = np.arange(count) * every
    steps[at] = r.integers(600, 900, count) * np.where(np.arange(count) % 2, 1, -1)  # past the code range
    x = (np.cumsum(steps) * 2e-3).astype(np.float32)
    c = ctx.compress(torch.from_numpy(x).cuda(), 1e-3, mode=fz.EB_ABS)
    y = ctx.decompress(c).cpu().numpy()
    ref = np.asarray(oracle.decompress(c.cpu().numpy().tobytes()), np.float32).reshape(-1)
    assert np.array_equal(y.view(np.uint32), ref.view(np.uint32))
