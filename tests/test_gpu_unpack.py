"""Byte masks: widths around the 16-byte pieces of the unpacking kernel and
outputs at every alignment (a piece that crosses a row end, the unaligned head
and tail), single and batched; and the atoms' short tasks next to their long
ones.  Packed masks of the same call are the reference, and the oracle theirs."""
import numpy as np
import pytest

import oracle
import paper_2010_07284_amd as vlg

pytestmark = pytest.mark.gpu

SRC = 'let a = intensity(img) >. 0.5\noutput "a" a\noutput "n" near(a) & !a'


@pytest.mark.parametrize("h,w", [(1, 1), (3, 5), (7, 15), (5, 16), (9, 17), (4, 63), (3, 64), (6, 65), (2, 1000),
                                 (33, 129), (130, 4001)])
def test_unpack_shapes_and_alignments(h, w):
    import torch
    ctx = vlg.create()
    img = np.random.default_rng([h, w]).random((1, h, w)).astype(np.float32)
    want = oracle.run(SRC, img)
    im, f = vlg.load_image(ctx, img), vlg.compile_formula(ctx, SRC)
    for off in (0, 1, 7, 15):
        buf = torch.full((2 * h * w + 64,), 7, dtype=torch.uint8, device="cuda")
        outs = [buf[off + k * h * w: off + (k + 1) * h * w].view(h, w) for k in range(2)]
        vlg.check_all(ctx, f, im, outs, fmt="u8")
        vlg.check_batch(ctx, f, [im], [[o.clone().fill_(9) for o in outs]], fmt="u8")
        vlg.sync(ctx)
        for o, x in zip(outs, want):
            assert np.array_equal(o.cpu().numpy(), x), off
        rest = buf.cpu().numpy()
        assert (rest[:off] == 7).all() and (rest[off + 2 * h * w:] == 7).all()


def test_batched_unpack_skips_and_offsets():
    import torch
    ctx = vlg.create()
    rng = np.random.default_rng(5)
    imgs = [rng.random((1, h, w)).astype(np.float32) for h, w in [(5, 7), (64, 64), (33, 250), (1, 1)]]
    ims, f = [vlg.load_image(ctx, x) for x in imgs], vlg.compile_formula(ctx, SRC)
    buf = torch.full((sum(2 * x[0].size for x in imgs) + 3,), 7, dtype=torch.uint8, device="cuda")
    at, outs = 3, []
    for x in imgs:
        h, w = x.shape[1:]
        outs.append([buf[at + k * h * w: at + (k + 1) * h * w].view(h, w) for k in range(2)])
        at += 2 * h * w
    outs[1][0] = None
    vlg.check_batch(ctx, f, ims, outs, fmt="u8")
    vlg.sync(ctx)
    for x, row in zip(imgs, outs):
        for o, want in zip(row, oracle.run(SRC, x)):
            if o is not None:
                assert np.array_equal(o.cpu().numpy(), want)
    assert (buf[3 + 70: 3 + 70 + 4096].cpu().numpy() == 7).all()  # the skipped output


@pytest.mark.parametrize("h,w", [(1, 1000), (63, 64), (1025, 33), (2048, 4096), (2047, 4100)])
@pytest.mark.parametrize("dtype", ["float32", "uint8", "uint16"])
def test_atom_tasks(h, w, dtype):
    ctx = vlg.create()
    top = {"float32": 1.0, "uint8": 255, "uint16": 65535}[dtype]
    img = (np.random.default_rng(h + w).random((1, h, w)) * top).astype(dtype)
    src = f'output "a" intensity(img) >. {0.25 * top}\noutput "b" intensity(img) <=. {0.75 * top}'
    im, f = vlg.load_image(ctx, img), vlg.compile_formula(ctx, src)
    got = vlg.check_all(ctx, f, im)
    vlg.sync(ctx)
    x = img[0].astype(np.float32)
    assert np.array_equal(vlg.unpack(got[0], h, w), x > np.float32(0.25 * top))
    assert np.array_equal(vlg.unpack(got[1], h, w), x <= np.float32(0.75 * top))
