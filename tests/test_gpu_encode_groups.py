"""Containers against the oracle at the tile counts where the encoder's
grouping changes (1, 4 and 8 tiles of 4 blocks per workgroup), with ragged
last tiles, and a rejected bound after a call that left other data in the
codes' buffer."""
import numpy as np
import pytest
import torch

import oracle
from inputs import fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1, 2, 255, 256, 257, 259, 6143, 6144, 6145, 6151])
def test_group_edges(fz, tiles):
    ctx = fz.Context(0)
    n = 2048 * tiles - 513
    x = fields.sorted_positions(n, seed=tiles)
    c = ctx.compress(torch.from_numpy(x).cuda(), 1e-5).cpu().numpy().tobytes()
    assert c == oracle.compress(x, 1e-5, 1)


def test_rejected_bound_after_shuffle(fz):
    ctx = fz.Context(0)
    x = torch.from_numpy(fields.random_small((64, 64, 64), seed=3, kind="smooth")).cuda()
    a = ctx.compress(x, 1e-3)
    for _ in range(2):
        ctx.compress(x, 1e-5, codec="shuffle")
        with pytest.raises(fz.FZError) as e:
            ctx.compress(x * 1e-30, 1e-299)
        assert e.value.code == -2
    assert torch.equal(ctx.compress(x, 1e-3), a)
