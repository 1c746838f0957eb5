"""Fused segments at the edges of their tiles and windows: images around one
and two words wide and around the 64 - 2 * halo rows that a tile stores, near
chains as deep as the halo, complements and constants as operands, against
the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2010_07284_amd as vlg
from tests.gpu_util import assert_same, gpu_run

pytestmark = pytest.mark.gpu


def source(depth):
    lines = ["let a0 = intensity(img, 0) >. 0.97", "let b = intensity(img, 1) >. 0.3", "let c = intensity(img, 1) <. 0.02"]
    for k in range(depth):  # dilations and erosions in turn, cut by b and c
        op = ("near(a%d)", "near(a%d) & b", "!near(!a%d | c)", "near(a%d & !c) | c")[k % 4] % k
        lines.append("let a%d = %s" % (k + 1, op))
    return "\n".join(lines + ['output "x" a%d' % depth, 'output "y" a%d & !b' % (depth // 2), 'output "z" !near(!a%d)' % (depth - 2)])


@pytest.fixture(scope="module")
def ctx():
    return vlg.create()


@pytest.mark.parametrize("halo", [2, 4, 8, 16])
def test_window_edges(ctx, halo):
    rng = np.random.default_rng(halo)
    src = source(halo)
    vlg.set_tunable(ctx, "fuse_halo", halo)
    try:
        for h in (1, 15, 17, 33, 64 - 2 * halo + 1):
            for w in (1, 63, 64, 65, 128, 161):
                img = rng.random((2, h, w)).astype(np.float32)
                assert_same(src, img, gpu_run(ctx, src, img, "fused"), oracle.run(src, img), tag=f"halo={halo} {h}x{w}")
    finally:
        vlg.set_tunable(ctx, "fuse_halo", 0)
