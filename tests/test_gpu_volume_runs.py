"""The volume labelling at the edges of its tiles (16 slices x 16 rows x 128
columns): sides around them, thin volumes, densities around and far above the
percolation threshold; one user of a labelling and several, single voxels
that join tiles only across a face, an edge or a corner.  Masks and labels are
compared with the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2010_07284_amd as vlg

pytestmark = pytest.mark.gpu

SRC = """
let a = intensity(img, 0) >. 0.995
let b = intensity(img, 1) >. 0.5
let c = intensity(img, 0) <. 0.01
output "g1" grow(a, b)
output "g2" grow(c, b)
output "g3" reach(c, b)
output "s1" surrounded(b, c)
output "g4" grow(c, !b)
"""
SHAPES = [(15, 17, 127), (16, 16, 128), (17, 15, 129), (33, 34, 257), (1, 35, 300), (40, 1, 260), (34, 33, 2),
          (18, 50, 63)]


@pytest.fixture(scope="module")
def ctx():
    return vlg.create()


def run(ctx, vol):
    C, D, H, W = vol.shape
    outs = vlg.check_all(ctx, vlg.compile_formula(ctx, SRC), vlg.load_volume(ctx, vol))
    vlg.sync(ctx)
    return [vlg.unpack(o, D * H, W).reshape(D, H, W) for o in outs]


def labels(ctx, m):
    import torch
    D, H, W = m.shape
    lab = vlg.ccl_labels3(ctx, torch.from_numpy(vlg.pack(m.reshape(D * H, W))).cuda(), D, H, W)
    vlg.sync(ctx)
    return lab.cpu().numpy().reshape(D, H, W)


@pytest.mark.parametrize("shape", SHAPES)
def test_tile_edges(ctx, shape):
    rng = np.random.default_rng(sum(shape))
    for p in (0.03, 0.1, 0.4):
        m = rng.random(shape) < p
        m[::3, ::2] |= rng.random(shape)[::3, ::2] < 4 * p  # some longer runs
        vol = np.stack([rng.random(shape), m]).astype(np.float32)
        for k, (got, want) in enumerate(zip(run(ctx, vol), oracle.run3(SRC, vol))):
            assert np.array_equal(got, want), (shape, p, k)
        assert np.array_equal(labels(ctx, m.astype(np.uint8)), oracle.ccl3(m.astype(np.uint8)).reshape(shape)), (shape, p)


def test_contacts_across_tiles(ctx):
    """Two voxels on both sides of a tile corner, in all 13 directions: one
    component each, the second voxel reached from the first."""
    for dz, dy, dx in [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1) if (a, b, c) > (0, 0, 0)]:
        m = np.zeros((20, 20, 132), np.uint8)
        p = (15 if dz > 0 else 9, 15 if dy > 0 else 16 if dy < 0 else 9, 127 if dx > 0 else 128 if dx < 0 else 90)
        q = (p[0] + dz, p[1] + dy, p[2] + dx)
        m[p] = m[q] = 1
        lab = labels(ctx, m)
        assert lab[p] == lab[q] == oracle.ccl3(m).reshape(m.shape)[p] and (lab >= 0).sum() == 2, (dz, dy, dx)
