"""The paper's labelling at the edges of its waves (four rows of 64 columns)
and of its row loads (images narrower than, as wide as and wider than the
three labels of a load): labels and iterations of the oracle's run, for
reconnects after fewer and after more iterations than are enqueued ahead of
the termination check; reachability with the seeds on those edges."""
import numpy as np
import pytest

import oracle
import paper_2010_07284_amd as vlg
from tests.gpu_util import assert_same, gpu_run

pytestmark = pytest.mark.gpu

SIDES = [1, 2, 3, 4, 5, 63, 64, 65, 129]


@pytest.fixture(scope="module")
def ctx():
    return vlg.create()


@pytest.mark.parametrize("k", [3, 5])
def test_labels_and_iterations(ctx, k):
    import torch
    for h in SIDES[:7]:
        for w in SIDES:
            m = (np.random.default_rng([h, w]).random((h, w)) < 0.6).astype(np.uint8)
            want, iters = oracle.ccl_pj(m, k=k)
            lab, st = vlg.ccl_labels_pj(ctx, torch.from_numpy(vlg.pack(m)).cuda(), h, w, k)
            vlg.sync(ctx)
            assert np.array_equal(lab.cpu().numpy(), want) and st["main_iterations"] == iters, (h, w)


def test_reach(ctx):
    src = ('let a = intensity(img, 0) >. 0.9\nlet b = intensity(img, 1) >. 0.45\n'
           'output "g" grow(a, b)\noutput "r" reach(b & a, b)\noutput "s" surrounded(b, a)\n')
    vlg.set_tunable(ctx, "ccl_algo", vlg.CCL_POINTER_JUMPING)
    try:
        for h, w in [(3, 65), (4, 64), (5, 129), (66, 3), (9, 2)]:
            img = np.random.default_rng([h, w, 1]).random((2, h, w)).astype(np.float32)
            assert_same(src, img, gpu_run(ctx, src, img, "fused"), oracle.run(src, img), tag=f"{h}x{w}")
    finally:
        vlg.set_tunable(ctx, "ccl_algo", 0)
