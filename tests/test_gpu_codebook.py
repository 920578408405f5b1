"""The device's code lengths against the oracle's package-merge at the edges
of its sort and merges: numbers of used codes around powers of two, equal
counts, counts that make the length limit bind, and a field of more than
2^32 / 12 values, whose weights take 64 bits."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fz):
    return fz.Context(0)


def _lens(c):
    p = np.frombuffer(c, np.uint8)[128:640]
    out = np.zeros(1024, np.uint8)
    out[0::2] = p & 15
    out[1::2] = p >> 4
    return out


def _field(counts):
    """1D field (absolute bound 0.5) whose residuals take the k-th value
    counts[k] times, except each block's first, which is 0."""
    vals = np.concatenate([np.full(int(c), k, np.int64) for k, c in enumerate(counts)])
    vals = np.where(vals % 2 == 1, (vals + 1) // 2, -(vals // 2))
    r = np.random.default_rng(len(vals))
    r.shuffle(vals)
    pad = (-len(vals)) % 511
    vals = np.concatenate([vals, np.zeros(pad, np.int64)]).reshape(-1, 511)
    x = np.zeros((vals.shape[0], 512), np.int64)
    x[:, 1:] = np.cumsum(vals, axis=1)
    return x.reshape(-1).astype(np.float32)


CASES = {f"equal{n}": np.full(n, 3) for n in (2, 3, 63, 64, 65, 127, 128, 129, 255, 257, 511, 513, 1000, 1023)}
CASES["fibonacci"] = np.array([1, 1, 2, 3, 5, 8, 13, 21, 34, 55, 89, 144, 233, 377, 610, 987, 1597, 2584])[::-1]
CASES["powers"] = np.array([2 ** k for k in range(16)])[::-1]
CASES["laplace"] = np.maximum(1, (40000 * np.exp(-np.arange(1023) / 60)).astype(int))
CASES["ties"] = np.repeat([64, 32, 8, 7, 1], [1, 30, 200, 200, 500])


@pytest.mark.parametrize("name", list(CASES))
def test_code_lengths(fz, ctx, name):
    x = _field(CASES[name])
    c = ctx.compress(torch.from_numpy(x).cuda(), 0.5, 0).cpu().numpy().tobytes()
    assert c == oracle.compress(x, 0.5, 0)


def test_weights_of_64_bits(fz, ctx):
    n = 2 ** 32 // 12 + 512 * 1000
    x = torch.zeros(n, dtype=torch.float32, device="cuda")
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x[::37] = (torch.randn((n + 36) // 37, generator=g, device="cuda") * 120).clamp_(-500, 500)
    c = ctx.compress(x, 0.5, 0)[:640].cpu().numpy().tobytes()
    hist = ctx.last_histogram()
    assert int(hist.astype(np.uint64).sum()) == n
    assert np.array_equal(_lens(c), oracle.codebook(hist))
