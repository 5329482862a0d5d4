"""What lets a layer that keeps the order of its sums take any tile for an undivided product: a channel of a convolution has the
same bits whichever tile computes it.  The same filters alone and among further ones, for which the plan has another tile, 256 x 64
or 256 x 160 against 128 x 128 or 256 x 256, or the same at another width; undivided both."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K
from test_gpu_conv_broad import g      # noqa: F401


SQUARE, LARGE, BROAD, SLIM = K.PRODUCT_SMALL, K.PRODUCT_LARGE, K.PRODUCT_BROAD, K.PRODUCT_NARROW


@pytest.mark.parametrize("n,h,ci,co,more,k,stride,on", [(25, 113, 24, 64, 128, 3, 1, (SLIM, SQUARE)), (25, 113, 24, 40, 256, 3, 1, (SLIM, LARGE)), (11, 113, 8, 64, 128, 7, 2, (SLIM, SQUARE)),
                                                        (43, 31, 8, 24, 128, 3, 1, (SLIM, SQUARE)), (64, 31, 40, 152, 512, 3, 1, (BROAD, LARGE)), (14, 98, 40, 152, 256, 3, 2, (LARGE, LARGE)),
                                                        (28, 30, 56, 152, 1024, 3, 1, (SQUARE, LARGE)), (16, 33, 64, 64, 128, 3, 1, (SQUARE, SQUARE)), (9, 65, 8, 48, 256, 7, 2, (SQUARE, SQUARE)),
                                                        (65, 30, 320, 160, 1024, 1, 1, (SQUARE, SQUARE))])
def test_same_bits(g, n, h, ci, co, more, k, stride, on):      # noqa: F811
    import torch
    plans = [K.conv_plan(K.ConvShape(n, h, h, ci, c, k, k, stride, k // 2), K.CONV_FWD | K.CONV_KEEP_SUMS | K.PLAN_TILES) for c in (co, more)]
    assert [(p[0][0], p[0][3]) for p in plans] == [(kernel, 1) for kernel in on]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + co)
    make = lambda *shape: torch.randn(shape, device="cuda", generator=gen).bfloat16()
    o, pad = (h + 2 * (k // 2) - k) // stride + 1, k // 2
    x, w = make(n, h, h, ci), make(more, k, k, ci)

    def forward(channels):
        y = torch.empty((n, o, o, channels), dtype=torch.bfloat16, device="cuda")
        part = w[:channels].contiguous()
        shape = K.binding.ConvShape(n, h, h, ci, channels, k, k, stride, pad)
        g.call(K.lib().karma_k_conv2d_fwd_bf16, g.ptr(x), g.ptr(part), g.ptr(y), C.byref(shape), g.stream_ptr())
        torch.cuda.synchronize()
        return y

    assert torch.equal(forward(co), forward(more)[..., :co])
