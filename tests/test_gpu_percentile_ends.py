"""Percentiles near the lowest and the highest rank of channels with so many
pixels that an open bracket (one that reaches the end of the sample) holds
more than 65536 candidates: their digits are then counted by many workgroups.
float32 and uint16, with and without ties at the end, single and batched, as
in test_gpu_percentile_sampled."""
import numpy as np
import pytest

from tests.test_gpu_percentile_sampled import check

pytestmark = pytest.mark.gpu

TOP = (0.9985, 0.999, 0.9995, 1.0)
LOW = (0.0, 0.0004, 0.0011, 0.002)


def channel(kind, shape, dtype):
    rng = np.random.default_rng([len(kind), shape[0]])
    x = rng.random(shape, dtype=np.float32)
    if kind == "levels":      # 256 distinct values
        x = np.floor(x * 256) / np.float32(255.99)
    elif kind == "ends":      # a few tenths of a percent at either end
        r = rng.random(shape, dtype=np.float32)
        x[r < 0.003] = 0.0
        x[r > 0.997] = 1.0
    if dtype == "float32":
        return x * np.float32(3) - np.float32(1)
    return np.round(x * np.float32(65535)).astype(dtype)


@pytest.mark.parametrize("dtype", ["float32", "uint16"])
@pytest.mark.parametrize("kind,shape", [("spread", (5200, 5000)), ("ends", (5200, 5000)), ("levels", (4099, 4200))])
def test_open_brackets(kind, shape, dtype):
    img = channel(kind, shape, dtype)
    for qs in (TOP, LOW):  # (four ranks of a large uint16 image take the radix select)
        check(img, qs[:2])
        check(img, qs[2:])
