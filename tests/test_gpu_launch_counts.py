"""Launches of a labelling as vlg_ccl_read_counters and vlg_formula_info report
them: one tile or several, one user or several, launched step by step, replayed
from a graph, batched, on volumes, and for the label calls."""
import numpy as np
import pytest

import paper_2010_07284_amd as vlg

pytestmark = pytest.mark.gpu

ATOMS = "let a = intensity(img) >. 200\nlet b = intensity(img) >. 100\nlet c = intensity(img) >. 220\n"
ONE = ATOMS + 'output "x" reach(a, b)'
TWO = ATOMS + 'output "x" reach(a, b)\noutput "y" reach(c, b)'


def launches(ctx):
    return vlg.ccl_counters(ctx)["launches_per_ccl"]


def test_counts():
    import torch
    ctx = vlg.create()
    assert launches(ctx) == 0
    one, two, none = (vlg.compile_formula(ctx, s) for s in (ONE, TWO, ATOMS + 'output "x" a | c'))
    rng = np.random.default_rng(1)
    for shape, merges in (((10, 100), 0), ((300, 400), 1)):
        im = vlg.load_image(ctx, rng.integers(0, 256, shape, dtype=np.uint8))
        for mode in ("fused", "graph", "graph"):
            vlg.set_mode(ctx, mode)
            for f, want in ((one, 2 + merges), (two, 2 + 2 * merges), (one, 2 + merges), (none, 2 + merges)):
                vlg.check_all(ctx, f, im)
                assert launches(ctx) == want, (shape, mode)
        for f, want in ((two, 4), (one, 3)):
            vlg.check_batch(ctx, f, [im, im])
            assert launches(ctx) == want
        mask = torch.from_numpy(vlg.pack((rng.random(shape) < 0.5).astype(np.uint8))).cuda()
        vlg.ccl_labels(ctx, mask, *shape)
        assert launches(ctx) == 2 + 2 * merges
    for shape, merges in (((4, 10, 60), 0), ((20, 10, 60), 1)):
        vol = vlg.load_volume(ctx, rng.integers(0, 256, shape, dtype=np.uint8))
        for f, want in ((one, 2 + merges), (two, 3 + merges)):
            vlg.check_all(ctx, f, vol)
            assert launches(ctx) == want, shape
        vlg.ccl_labels3(ctx, torch.zeros((shape[0] * shape[1], 1), dtype=torch.int64, device="cuda"), *shape)
        assert launches(ctx) == 3 + merges


def test_graph_without_labelling():
    """Its replay leaves the count of the last labelling as it is."""
    ctx = vlg.create()
    one, two, none = (vlg.compile_formula(ctx, s) for s in (ONE, TWO, ATOMS + 'output "x" a | c'))
    im = vlg.load_image(ctx, np.random.default_rng(2).integers(0, 256, (300, 400), dtype=np.uint8))
    vlg.set_mode(ctx, "graph")
    # (`two` first: the workspace, and with it the graphs, stays)
    calls = ((two, 4), (none, 4), (one, 3), (none, 3), (two, 4), (none, 4))
    outs = {f: vlg.check_all(ctx, f, im) for f in (two, one, none)}
    for f, want in calls:
        vlg.check_all(ctx, f, im, outs=outs[f])
        assert launches(ctx) == want
    outs = {f: vlg.check_batch(ctx, f, [im, im]) for f in (two, one, none)}
    for f, want in calls:
        vlg.check_batch(ctx, f, [im, im], outs=outs[f])
        assert launches(ctx) == want


def test_formula_info():
    ctx = vlg.create()
    info = [vlg.formula_info(vlg.compile_formula(ctx, s)) for s in (ONE, TWO)]
    assert info[0]["launches_fused"] == info[0]["steps_fused"] - 1  # one user: no pass that flags the roots
    assert info[1]["launches_fused"] == info[1]["steps_fused"]
