"""Components that cross long rows and columns of tiles: every walk of the
labelling ends within 40 steps (a loop cap of 40 is never reached), whatever
the tile height and so the distance between the tiles' node ids.  Each line of
the mask is reached from its one end."""
import numpy as np
import pytest

import paper_2010_07284_amd as vlg

pytestmark = pytest.mark.gpu

SRC = """
let b = intensity(img, 0) >. 0
let s = intensity(img, 1) >. 0
let t = intensity(img, 2) >. 0
output "s" reach(s, b) & b
output "t" reach(t, b) & b
"""


def lines(h, w, vertical):
    """Every second row (or column), the first of them seeded at their start
    and the rest at their end."""
    img = np.zeros((3, h, w), np.uint8)
    m = img.transpose(0, 2, 1) if vertical else img
    m[0, ::2] = 1
    cut = m.shape[1] // 2
    m[1, :cut, 0] = 1
    m[2, cut:, -1] = 1
    m[1] &= m[0]
    m[2] &= m[0]
    want = np.zeros((2, h, w), np.uint8)
    k = want.transpose(0, 2, 1) if vertical else want
    k[0, :cut:2] = 1
    k[1, cut + cut % 2::2] = 1
    return img, want


@pytest.mark.parametrize("tile_rows", [8, 16, 32])
@pytest.mark.parametrize("h,w", [(64, 60000), (130, 20000), (20000, 130), (1024, 1024)])
def test_walks_stay_short(h, w, tile_rows):
    for vertical in (False, True):
        ctx = vlg.create()
        vlg.set_mode(ctx, "fused")
        vlg.set_tunable(ctx, "ccl_tile_rows", tile_rows)
        vlg.set_loop_cap(ctx, 40)
        img, want = lines(h, w, vertical)
        im, f = vlg.load_image(ctx, img), vlg.compile_formula(ctx, SRC)
        for outs in (vlg.check_all(ctx, f, im), vlg.check_batch(ctx, f, [im])[0]):
            vlg.sync(ctx)
            for k in range(2):
                assert np.array_equal(vlg.unpack(outs[k], h, w), want[k]), (vertical, k)
