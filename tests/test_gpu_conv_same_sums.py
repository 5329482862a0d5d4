"""What lets a layer that keeps the order of its sums take any tile for an undivided product: a channel of a convolution has the
same bits whichever tile computes it.  The same filters alone and among further ones, for which another tile is chosen."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K
from test_gpu_conv_broad import g      # noqa: F401


@pytest.mark.parametrize("n,h,ci,co,more,k,stride", [(16, 33, 64, 64, 128, 3, 1), (9, 65, 8, 48, 256, 7, 2), (64, 31, 40, 152, 512, 3, 1), (65, 30, 320, 160, 1024, 1, 1)])
def test_same_bits(g, n, h, ci, co, more, k, stride):      # noqa: F811
    import torch
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
