"""Labels of volumes of many small components, a run per block and up to 64
runs per row of a tile: lattices of single voxels, of lines along each axis,
sparse noise, and lattices beside one large component; whole tiles and ragged
ends.  Labels are compared with the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2010_07284_amd as vlg
from tests.test_gpu_volume_runs import labels

pytestmark = pytest.mark.gpu


def masks(shape):
    z, y, x = np.ogrid[:shape[0], :shape[1], :shape[2]]
    rng = np.random.default_rng(shape)
    even = (x % 2 == 0) & (y % 2 == 0)
    yield "voxels", even & (z % 2 == 0)
    yield "along z", even & (z >= 0)
    yield "along y", (x % 2 == 0) & (z % 2 == 0) & (y >= 0)
    yield "along x", (y % 2 == 0) & (z % 2 == 0) & (x >= 0)
    yield "noise", rng.random(shape) < 0.05
    big = even & (z % 2 == 0)
    big[:, :shape[1] // 2] |= rng.random((shape[0], shape[1] // 2, shape[2])) < 0.3
    yield "beside a large one", big
    yield "few per row", even & (z >= 0) & (x % 128 < 20)


@pytest.mark.parametrize("shape", [(32, 32, 128), (35, 18, 261), (3, 70, 127), (64, 64, 64)])
def test_labels(shape):
    ctx = vlg.create()
    for name, m in masks(shape):
        m = np.ascontiguousarray(m, dtype=np.uint8)
        assert np.array_equal(labels(ctx, m), oracle.ccl3(m).reshape(shape)), (shape, name)
