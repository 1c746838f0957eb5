"""Percentiles of channels whose candidates lie in a few rows of each period, and
of channels made so that every bracket misses its rank or holds most pixels:
the same values as a sort gives, in at most three (periodic) or eight times
the time of noise of the same size (one workgroup selecting over the whole
channel takes over a hundred times as long)."""
import time

import numpy as np
import pytest

import paper_2010_07284_amd as vlg
from tests.test_gpu_percentile_sampled import check, sampled_places

pytestmark = pytest.mark.gpu


def sine(period, shape, dtype):
    rng = np.random.default_rng(period)
    x = (0.5 + 0.4 * np.sin(np.arange(shape[0], dtype=np.float32) * np.float32(2 * np.pi / period)))[:, None] + \
        0.1 * (rng.random(shape, dtype=np.float32) - np.float32(0.5))
    return typed(x, dtype)


def typed(x, dtype):
    return x.astype(np.float32) if dtype == "float32" else np.round(x * 65535).astype(dtype)


def time_of(img, qs):
    import torch
    ctx = vlg.create()
    f = vlg.compile_formula(ctx, "\n".join(f'output "o{k}" intensity(img) >. percentile(img, 0, {q})'
                                           for k, q in enumerate(qs)))
    im = vlg.load_image(ctx, img)
    outs = vlg.check_all(ctx, f, im)
    best = 1e9
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(4):
            vlg.check_all(ctx, f, im, outs)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("dtype", ["float32", "uint16"])
@pytest.mark.parametrize("shape", [(4096, 4096), (2048, 2048), (3000, 5000)])
def test_periodic_rows(shape, dtype):
    noise = typed(np.random.default_rng(1).random(shape, dtype=np.float32), dtype)
    limit = {qs: 3 * time_of(noise, qs) for qs in ((0.5,), (0.95, 0.86))}
    for period in (8, 16, 32, 64, 256):
        img = sine(period, shape, dtype)
        check(img, (0.5, 0.95, 0.86))
        for qs, most in limit.items():
            assert time_of(img, qs) < most, (period, qs)


@pytest.mark.parametrize("dtype", ["float32", "uint16"])
@pytest.mark.parametrize("shape", [(4096, 4096), (1999, 3001)])
def test_channels_that_the_sample_misjudges(shape, dtype):
    rng = np.random.default_rng(shape)
    n, at = shape[0] * shape[1], sampled_places(shape[0] * shape[1])
    noise = rng.random(shape, dtype=np.float32)
    qs = (0.5, 0.9)
    limit = 8 * time_of(typed(noise, dtype), qs)
    missed = noise.reshape(-1).copy()
    missed[at] = 0.25 + 0.0001 * rng.random(len(at), dtype=np.float32)
    flooded = (0.5 + 0.001 * noise).reshape(-1)  # one place in the order of the samples, most pixels in their bracket
    flooded[at] = rng.random(len(at), dtype=np.float32)
    ties = np.where(noise < 0.3, noise, np.float32(0.5)).reshape(-1)
    ties[at] = rng.random(len(at), dtype=np.float32)
    for name, x in (("missed", missed), ("flooded", flooded), ("ties", ties)):
        img = typed(x.reshape(shape), dtype)
        check(img, qs)
        assert time_of(img, qs) < limit, name
