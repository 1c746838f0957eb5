"""Several users of one labelling on masks of up to 64 runs per row of a tile:
lattices, lines, a comb that joins every line, sparse and dense noise, and
rows with a few runs only; single images, regions and batches, compared with
the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2010_07284_amd as vlg

pytestmark = pytest.mark.gpu

SRC = """
let b = intensity(img, 0) >. 0
let s = intensity(img, 1) >. 0
let t = intensity(img, 1) >. 1
output "r" reach(s, b)
output "t" grow(t, b)
output "i" reach(interior(s), b)
output "c" reach(s & b, b)
output "n" reach(t & near(b), b) & b
output "u" surrounded(b, s)
"""


def masks(h, w):
    y, x = np.ogrid[:h, :w]
    rng = np.random.default_rng([h, w])
    yield "voxels", (x % 2 == 0) & (y % 2 == 0)
    yield "columns", (x % 2 == 0) & (y >= 0)
    yield "comb", (x % 2 == 0) | (y == h - 1)
    yield "sparse", rng.random((h, w)) < 0.05
    yield "dense", rng.random((h, w)) < 0.5
    for n in (5, 9, 13, 33):  # runs per row of a tile around the loads' groups
        yield f"{n} runs", (x % 2 == 0) & (x % 128 < 2 * n) & (y >= 0)


@pytest.mark.parametrize("h,w", [(40, 64), (129, 260), (260, 131)])
def test_users(h, w):
    ctx = vlg.create()
    f = vlg.compile_formula(ctx, SRC)
    for k, (name, m) in enumerate(masks(h, w)):
        rng = np.random.default_rng(k)
        img = np.stack([m, (rng.random((h, w)) < 0.1) + (rng.random((h, w)) < 0.01)]).astype(np.uint8)
        want = oracle.run(SRC, img)
        im = vlg.load_image(ctx, img)
        for mode, lanes in (("fused", 1), ("graph", 4), ("perop", 1)):
            vlg.set_mode(ctx, mode)
            vlg.set_tunable(ctx, "ccl_lanes", lanes)
            for outs in (vlg.check_all(ctx, f, im), vlg.check_batch(ctx, f, [im])[0]):
                vlg.sync(ctx)
                for o, x in zip(outs, want):
                    assert np.array_equal(vlg.unpack(o, h, w), x), (name, mode)
