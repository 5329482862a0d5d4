"""Convolutions of a size at which the tile of 256 pixels x 160 channels (weight gradients 160 x 256) is modelled to be the
shortest: channels just below a tile and just above, images whose pixels are no whole tiles, stride 2 (the input gradient by
parity, whose four products differ in size on odd images), divided reductions.  Against the unfolded product in fp32.
The plan says which tile each of the three products is on.
A bf16 result carries one rounding (2^-9 per element); fp32 sums add less than that at these lengths."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def close(got, want, scale):
    return ((got.float() - want).abs() <= 2.0 ** -8 * want.abs() + 2e-5 * scale).all().item()


def tiles(n, h, ci, co, k, stride):
    """The tile each product is on: forward, input gradient, weight gradient with the workspace that check passes."""
    shape, room = K.ConvShape(n, h, h, ci, co, k, k, stride, k // 2), 64 * co * k * k * ci * 4
    parts = [K.conv_plan(shape, which | K.PLAN_TILES, room if which == K.CONV_WGRAD else 0) for which in (K.CONV_FWD, K.CONV_DGRAD, K.CONV_WGRAD)]
    assert all(len(p) == 1 for p in parts)
    return [p[0][0] for p in parts]


SQUARE, LARGE, BROAD, SLIM, FLAT = K.PRODUCT_SMALL, K.PRODUCT_LARGE, K.PRODUCT_BROAD, K.PRODUCT_NARROW, K.PRODUCT_FLAT


@pytest.mark.parametrize("n,h,ci,co,k,stride,on", [(64, 31, 40, 152, 3, 1, [BROAD, SLIM, SQUARE]), (64, 31, 280, 152, 3, 1, [BROAD, BROAD, BROAD]),
                                                   (100, 50, 40, 160, 3, 2, [BROAD, SLIM, SQUARE]), (128, 33, 152, 24, 3, 2, [SLIM, SQUARE, FLAT]), (36, 61, 160, 160, 5, 2, [BROAD, BROAD, BROAD]),
                                                   (65, 30, 312, 320, 1, 1, [SQUARE, SQUARE, SQUARE]), (61, 32, 160, 168, 3, 1, [LARGE, BROAD, FLAT]),
                                                   (37, 30, 152, 88, 3, 1, [SQUARE, BROAD, SQUARE]), (30, 54, 88, 160, 3, 1, [SQUARE, SQUARE, BROAD]),
                                                   (40, 51, 64, 160, 7, 2, [SQUARE, SLIM, BROAD])])
def test_forward_and_gradients(g, n, h, ci, co, k, stride, on):
    assert tiles(n, h, ci, co, k, stride) == on
    check(g, n, h, ci, co, k, stride)


def check(g, n, h, ci, co, k, stride):
    import torch
    F = torch.nn.functional
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n + h + ci)
    make = lambda *shape: torch.randn(shape, device="cuda", generator=gen).bfloat16()
    o, pad = (h + 2 * (k // 2) - k) // stride + 1, k // 2
    x, w, dy = make(n, h, h, ci), make(co, k, k, ci), make(n, o, o, co)
    shape = K.binding.ConvShape(n, h, h, ci, co, k, k, stride, pad)
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(w)
    wt, ws = torch.empty(w.numel(), dtype=torch.bfloat16, device="cuda"), torch.empty(64 * w.numel(), device="cuda")
    lib, s = K.lib(), C.byref(shape)
    g.call(lib.karma_k_conv2d_fwd_bf16, g.ptr(x), g.ptr(w), g.ptr(y), s, g.stream_ptr())
    g.call(lib.karma_k_conv2d_wgrad_bf16, g.ptr(dy), g.ptr(x), g.ptr(dw), g.ptr(ws), C.c_uint64(ws.numel() * 4), s, g.stream_ptr())
    g.call(lib.karma_k_conv2d_dgrad_bf16, g.ptr(dy), g.ptr(w), g.ptr(wt), None, g.ptr(dx), s, g.stream_ptr())
    rows = lambda t: F.unfold(t.float().permute(0, 3, 1, 2), k, padding=pad, stride=stride).permute(0, 2, 1).reshape(n * o * o, ci * k * k)
    wm = w.float().permute(0, 3, 1, 2).reshape(co, ci * k * k)
    cols, d = rows(x), dy.float().reshape(-1, co)
    assert close(y.reshape(-1, co), cols @ wm.t(), cols.abs() @ wm.abs().t())
    as_w = lambda m: m.reshape(co, ci, k, k).permute(0, 2, 3, 1)
    assert close(dw, as_w(d.t() @ cols), as_w(d.abs().t() @ cols.abs()))
    back = lambda a, b: F.fold((a @ b).reshape(n, o * o, ci * k * k).permute(0, 2, 1), (h, h), k, padding=pad, stride=stride).permute(0, 2, 3, 1)
    assert close(dx, back(d, wm), back(d.abs(), wm.abs()))
