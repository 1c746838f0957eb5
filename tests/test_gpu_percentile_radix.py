"""Four ranks of a uint16 channel around the size where they change from the
sampled to the radix select (2^22 pixels): values as a sort gives."""
import numpy as np
import pytest

from tests.test_gpu_percentile_sampled import check

pytestmark = pytest.mark.gpu

QS = (0.2, 0.9995, 0.6, 0.001)


@pytest.mark.parametrize("shape", [(2048, 2048), (2048, 2049), (1, 4194305), (3000, 3100)])
def test_values(shape):
    rng = np.random.default_rng(shape)
    for x in (rng.random(shape), np.where(rng.random(shape) < 0.4, 0.2, rng.random(shape))):
        check(np.round(x * 65535).astype(np.uint16), QS)

