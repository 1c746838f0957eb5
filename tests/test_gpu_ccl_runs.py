"""The run-based labelling at the edges of its tiles: image sides around the
tile width (128 pixels), the tile heights and the narrow or low images whose
tiles the workspace rule makes taller; one user of a labelling (components
with seeds united with the seed node) and several (flag and reseed passes),
one and several labellings per launch, single and batched.  Masks are
compared with the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2010_07284_amd as vlg
from tests.gpu_util import assert_same, gpu_run

pytestmark = pytest.mark.gpu

# one labelling of b with several users, then one with a single user each
SHARED = """
let a = intensity(img, 0) >. 0.9
let b = intensity(img, 1) >. 0.5
let c = intensity(img, 0) <. 0.08
let d = (intensity(img, 0) >. 0.4) & (intensity(img, 0) <. 0.43)
output "g1" grow(a, b)
output "g2" grow(c, b)
output "g3" reach(d, b)
output "s1" surrounded(b, c)
output "s2" grow(a & c, b)
output "g4" grow(c, !b)
"""
SHAPES = [(1, 1), (2, 129), (1, 1000), (1000, 1), (15, 127), (16, 128), (17, 129), (33, 131), (34, 258),
          (130, 3), (65, 640), (300, 66), (129, 257)]


def image(h, w, kind):
    rng = np.random.default_rng([h, w, 3])
    yy, xx = np.mgrid[:h, :w]
    b = {"noise": rng.random((h, w)) < 0.55, "columns": (xx % 2 == 0) | (rng.random((h, w)) < 0.02),
         "rows": (yy % 2 == 0) | (rng.random((h, w)) < 0.02)}[kind]
    return np.stack([rng.random((h, w)), b]).astype(np.float32)


@pytest.fixture(scope="module")
def ctx():
    return vlg.create()


@pytest.mark.parametrize("tbh", [8, 16, 32])
@pytest.mark.parametrize("kind", ["noise", "columns", "rows"])
def test_tile_edges(ctx, tbh, kind):
    vlg.set_tunable(ctx, "ccl_tile_rows", tbh)
    try:
        for h, w in SHAPES:
            img = image(h, w, kind)
            want = oracle.run(SHARED, img)
            for lanes in (1, 4):
                vlg.set_tunable(ctx, "ccl_lanes", lanes)
                assert_same(SHARED, img, gpu_run(ctx, SHARED, img, "fused"), want, tag=f"{h}x{w} lanes={lanes}")
    finally:
        vlg.set_tunable(ctx, "ccl_tile_rows", 0)
        vlg.set_tunable(ctx, "ccl_lanes", 0)


@pytest.mark.parametrize("tbh", [8, 32])
def test_tile_edges_batched(ctx, tbh):
    import torch
    vlg.set_tunable(ctx, "ccl_tile_rows", tbh)
    try:
        imgs = [image(h, w, k) for h, w in SHAPES for k in ("noise", "columns")]
        f = vlg.compile_formula(ctx, SHARED)
        got = vlg.check_batch(ctx, f, [vlg.load_image(ctx, torch.from_numpy(x).cuda()) for x in imgs])
        vlg.sync(ctx)
        for x, row in zip(imgs, got):
            for k, (o, want) in enumerate(zip(row, oracle.run(SHARED, x))):
                assert np.array_equal(vlg.unpack(o, *x.shape[1:]), want), (x.shape, k)
    finally:
        vlg.set_tunable(ctx, "ccl_tile_rows", 0)


def test_labels_of_narrow_images(ctx):
    import torch
    for h, w in SHAPES:
        m = image(h, w, "noise")[1].astype(np.uint8)
        lab = vlg.ccl_labels(ctx, torch.from_numpy(vlg.pack(m)).cuda(), h, w)
        vlg.sync(ctx)
        assert np.array_equal(lab.cpu().numpy(), oracle.ccl(m)), (h, w)


@pytest.mark.parametrize("tbh", [8, 16])
@pytest.mark.parametrize("h,w", [(1024, 1020), (1041, 1024), (1030, 1300)])
def test_rows_per_group(ctx, tbh, h, w):
    """Images on both sides of the line between groups of 16 and of 64 block rows."""
    vlg.set_tunable(ctx, "ccl_tile_rows", tbh)
    try:
        img = image(h, w, "noise")
        assert_same(SHARED, img, gpu_run(ctx, SHARED, img, "fused"), oracle.run(SHARED, img), tag=f"{h}x{w}")
    finally:
        vlg.set_tunable(ctx, "ccl_tile_rows", 0)
