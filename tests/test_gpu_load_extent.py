"""Device pixels whose declared shape reaches beyond their allocation: refused
with VLG_EHIP before any of them is read, while shapes that fit are loaded,
also after a refused one.  (The shapes tried end within the 4096 bytes that an
allocation occupies at least.)"""
import ctypes

import pytest

import paper_2010_07284_amd as vlg
from paper_2010_07284_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,es", [(1, 1), (2, 2), (0, 4)])
def test_rows_beyond_the_allocation(dtype, es):
    import torch
    torch.cuda.init()
    hip = ctypes.CDLL("libamdhip64.so")
    p = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(1200)) == 0
    ctx = vlg.create()

    def load(channels, h, w, pitch):
        out = ctypes.c_void_p()
        rc = _lib.lib().vlg_load_image(ctx.handle, p, dtype, channels, h, w, pitch, 1, ctypes.byref(out))
        vlg.sync(ctx)
        if rc == 0:
            _lib.call("vlg_image_free", out)
        return rc

    px = 1200 // es  # pixels that fit
    for shape in ((1, 1, px + 1, px + 1), (1, 1, px + 60, px + 60), (1, 3, px // 3 - 10, px // 3 + 10)):
        assert load(*shape) == -5
        for fits in ((1, 1, px, px), (2, 3, px // 6, px // 6), (1, 3, px // 3 - 10, px // 3)):
            assert load(*fits) == 0
    torch.cuda.synchronize()
    assert int(torch.ones(7, device="cuda").sum()) == 7  # no error is left for the next launch
    assert hip.hipFree(p) == 0
