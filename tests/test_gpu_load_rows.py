"""Loading device pixels: every pixel type, widths around the 16 bytes that a
lane writes and the 64 pixels of a word, sources at odd addresses and with
rows further apart than their width, and the ordering of the context's stream
against another one; checked through the masks of a comparison."""
import ctypes

import numpy as np
import pytest

import paper_2010_07284_amd as vlg

pytestmark = pytest.mark.gpu

SRC = 'output "a" intensity(img, 0) >. 0.5\noutput "b" intensity(img, 1) <=. 0.5\n'
TOP = {"float32": 1.0, "uint8": 255.0, "uint16": 65535.0}


@pytest.fixture(scope="module")
def ctx():
    return vlg.create()


@pytest.mark.parametrize("dtype", ["float32", "uint8", "uint16"])
@pytest.mark.parametrize("gap,start", [(0, 0), (0, 1), (3, 0), (5, 7)])
def test_rows(ctx, dtype, gap, start):
    import torch
    from paper_2010_07284_amd import _lib
    rng = np.random.default_rng(gap + start)
    src = SRC.replace("0.5", repr(0.5 * TOP[dtype]))
    f = vlg.compile_formula(ctx, src)
    for h, w in [(1, 1), (3, 4), (5, 15), (4, 16), (7, 17), (2, 63), (3, 64), (9, 65), (130, 200)]:
        pitch = w + gap
        flat = (rng.random(start + 2 * h * pitch) * TOP[dtype]).astype(dtype)
        dev = torch.from_numpy(flat.view(np.uint8)).cuda()
        torch.cuda.synchronize()
        out = ctypes.c_void_p()
        _lib.call("vlg_load_image", ctx.handle, ctypes.c_void_p(dev.data_ptr() + start * flat.itemsize),
                  {"float32": 0, "uint8": 1, "uint16": 2}[dtype], 2, h, w, pitch, 1, ctypes.byref(out))
        vlg.sync(ctx)
        im = vlg.Image(out, (2, h, w), None)
        img = flat[start:].reshape(2, h, pitch)[:, :, :w].astype(np.float32)
        t = np.float32(0.5 * TOP[dtype])
        a, b = (torch.zeros((h, (w + 63) // 64), dtype=torch.int64, device="cuda") for _ in range(2))
        vlg.check_all(ctx, f, im, [a, b])
        vlg.sync(ctx)
        assert np.array_equal(vlg.unpack(a, h, w), img[0] > t), (h, w)
        assert np.array_equal(vlg.unpack(b, h, w), img[1] <= t), (h, w)


def test_order_against_another_stream(ctx):
    """The masks written by a call are seen by work that torch enqueues after
    it, and the call waits for torch's pending writes to them."""
    import torch
    f = vlg.compile_formula(ctx, 'output "a" intensity(img) >. 0.5')
    img = np.random.default_rng(3).random((1, 700, 900)).astype(np.float32)
    im = vlg.load_image(ctx, img)
    want = torch.from_numpy(vlg.pack((img[0] > 0.5).astype(np.uint8))).cuda()
    side = torch.cuda.Stream()
    for stream in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(stream):
            for _ in range(20):
                out = torch.empty_like(want)
                big = torch.rand(1 << 22, device="cuda").sort()[0]  # keeps the stream busy
                out.fill_(-1)
                vlg.check_all(ctx, f, im, [out])
                assert bool((out == want).all()) and big.numel() > 0
