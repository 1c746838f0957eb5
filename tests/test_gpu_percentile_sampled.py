"""Percentiles by sampled brackets at the sizes where their steps change
(selection over the whole channel up to 32768 pixels, 8192, 12288 and 16384
samples, candidate segments), float32 and uint16, one to four ranks, with
ties of every weight; ranks that the brackets miss, forced by writing one
value at the sampled places; and NaN.  Values are pinned through a >= and a >
threshold, and compared with a sort of the keys."""
import numpy as np
import pytest

import paper_2010_07284_amd as vlg

pytestmark = pytest.mark.gpu

QS = (0.5, 0.95, 0.003, 0.86)


def nearest_rank(x, q):
    """The k-th smallest pixel by the order of the float32 bit patterns."""
    v = np.ascontiguousarray(x).reshape(-1)
    k = min(max(int(np.ceil(q * v.size)) - 1, 0), v.size - 1)
    if v.dtype != np.float32:
        return np.float32(np.partition(v, k)[k])
    u = v.view(np.uint32)
    key = np.where(u & 0x80000000, ~u, u | np.uint32(0x80000000))
    key = np.partition(key, k)[k]
    u = key & 0x7FFFFFFF if key & 0x80000000 else ~key
    return np.array([u], np.uint32).view(np.float32)[0]


def check(img, qs, mode="fused"):
    ctx = vlg.create()
    vlg.set_mode(ctx, mode)
    h, w = img.shape
    src = "\n".join(f'output "ge{k}" intensity(img) >=. percentile(img, 0, {q})\n'
                    f'output "gt{k}" intensity(img) >. percentile(img, 0, {q})' for k, q in enumerate(qs))
    f, im = vlg.compile_formula(ctx, src), vlg.load_image(ctx, img)
    single = vlg.check_all(ctx, f, im)
    batched = vlg.check_batch(ctx, f, [im])[0]
    vlg.sync(ctx)
    x = img.astype(np.float32)
    for k, q in enumerate(qs):
        v = nearest_rank(img, q)
        for got in (single, batched):
            assert np.array_equal(vlg.unpack(got[2 * k], h, w), x >= v), (img.shape, q, v)
            assert np.array_equal(vlg.unpack(got[2 * k + 1], h, w), x > v), (img.shape, q, v)


def values(rng, kind, shape, dtype):
    x = rng.random(shape)
    if kind == "half":      # half of the pixels equal, at the median's rank
        x[rng.random(shape) < 0.5] = 0.5
    elif kind == "light":   # ties a little lighter and a little heavier than a bracket
        x[rng.random(shape) < 0.04] = 0.501
        x[rng.random(shape) < 0.012] = 0.95
    elif kind == "floor":   # a constant background, brighter noise above
        x[rng.random(shape) < 0.7] = 0.0
    elif kind == "few":     # few distinct values
        x = np.round(x * 20) / 20
    if dtype == "float32":
        return (x * 2 - 0.5).astype(np.float32)
    return (x * 60000).astype(dtype)


SHAPES = [(181, 181), (1, 32769), (64, 513), (363, 361), (256, 513), (1449, 1450), (1, 200000), (70000, 3),
          (2048, 2051)]


@pytest.mark.parametrize("dtype", ["float32", "uint16"])
@pytest.mark.parametrize("kind", ["spread", "half", "light", "floor", "few"])
def test_steps(kind, dtype):
    rng = np.random.default_rng([len(kind), len(dtype)])
    for n, shape in enumerate(SHAPES):
        check(values(rng, kind, shape, dtype), QS[:1 + n % 4] if n % 2 else (0.0, 0.3, 1.0))


def sampled_places(n):
    """Flat pixel indices the brackets are sampled at."""
    sn = 8192 if n < 131072 else 12288 if n < 2 << 20 else 16384
    i = np.arange(sn, dtype=np.uint64)
    a, b = i * np.uint64(n) // np.uint64(sn), (i + np.uint64(1)) * np.uint64(n) // np.uint64(sn)
    m = np.uint64(0xFFFFFFFF)
    x = (i * np.uint64(0x9E3779B1)) & m
    x = ((x ^ (x >> np.uint64(15))) * np.uint64(0x85EBCA77)) & m
    x ^= x >> np.uint64(13)
    return (a + ((x * (b - a)) >> np.uint64(32))).astype(np.int64)


@pytest.mark.parametrize("shape", [(200, 301), (700, 1001), (2100, 2049)])
def test_missed_brackets(shape):
    # the samples all say 0.25, or all lie in a narrow range: the ranks of the
    # other pixels are outside every bracket
    rng = np.random.default_rng(shape)
    n = shape[0] * shape[1]
    for lo, hi in ((0.25, 0.25), (0.25, 0.2501)):
        x = rng.random(n).astype(np.float32)
        x[sampled_places(n)] = rng.uniform(lo, hi, len(sampled_places(n))).astype(np.float32)
        check(x.reshape(shape), (0.5, 0.9, 0.2))


def test_nan_and_infinities_keep_their_order():
    rng = np.random.default_rng(9)
    x = rng.standard_normal((600, 500)).astype(np.float32)
    for v, p in ((np.nan, 0.02), (-np.nan, 0.02), (np.inf, 0.03), (-np.inf, 0.03), (-0.0, 0.02)):
        x[rng.random(x.shape) < p] = v
    x.view(np.uint32)[rng.random(x.shape) < 0.002] = 0xFFFFFFFF
    x.view(np.uint32)[rng.random(x.shape) < 0.002] = 0x7FFFFFFF
    check(x, (0.06, 0.5, 0.93))
    check(x, (0.0, 1.0, 0.0001, 0.9999))


@pytest.mark.parametrize("dtype", ["float32", "uint16"])
@pytest.mark.parametrize("width", [0.0, 2e-6, 1e-4])
def test_crowded_bucket(dtype, width):
    # a twentieth of the pixels in one narrow range (or one value) within the
    # bracket of the median, whose ends lie far from it
    rng = np.random.default_rng(int(width * 1e7))
    x = rng.choice([0.02, 0.9], (2049, 2050)) + 0.08 * rng.random((2049, 2050))
    crowd = rng.random(x.shape) < 0.045
    x[crowd] = 0.5 + width * rng.random(int(crowd.sum()))
    x = (x * 2 - 0.5).astype(np.float32) if dtype == "float32" else (x * 60000).astype(dtype)
    check(x, (0.49, 0.5, 0.505))
