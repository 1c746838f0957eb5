"""N on word columns packed across bands: widths around one, two and 64 words,
heights around the band heights, every band height, single images and a batch;
complements (padding bits) included, against the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2010_07284_amd as vlg
from tests.gpu_util import assert_same, gpu_run

pytestmark = pytest.mark.gpu

SRC = """
let a = intensity(img, 0) >. 0.98
let b = intensity(img, 1) >. 0.5
output "n" near(a)
output "i" interior(b)
output "o" near(!b) | a
output "x" !near(a & b) & b
output "nn" near(near(!a & b))
"""
SIZES = [(1, 1), (3, 64), (4, 65), (5, 63), (8, 129), (9, 700), (31, 70), (33, 4100), (65, 4032), (130, 200)]


@pytest.fixture(scope="module")
def ctx():
    return vlg.create()


def images():
    rng = np.random.default_rng(12)
    return [rng.random((2, h, w)).astype(np.float32) for h, w in SIZES]


@pytest.mark.parametrize("rows", [4, 8, 16, 32])
def test_single(ctx, rows):
    vlg.set_tunable(ctx, "near_band_rows", rows)
    try:
        for img in images():
            want = oracle.run(SRC, img)
            for mode in ("perop", "fused"):
                assert_same(SRC, img, gpu_run(ctx, SRC, img, mode), want, tag=f"{mode} {rows} {img.shape}")
    finally:
        vlg.set_tunable(ctx, "near_band_rows", 0)


def test_batch(ctx):
    imgs = images()
    f = vlg.compile_formula(ctx, SRC)
    outs = vlg.check_batch(ctx, f, [vlg.load_image(ctx, i) for i in imgs])
    vlg.sync(ctx)
    for img, got in zip(imgs, outs):
        got = [vlg.unpack(o, *img.shape[1:]) for o in got]
        assert_same(SRC, img, got, oracle.run(SRC, img), tag=f"batch {img.shape}")
