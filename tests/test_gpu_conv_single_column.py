"""Convolutions whose output is one pixel wide, or whose filter is one tap wide and several high: where a kernel divides by the
width through a reciprocal, the reciprocal of one does not fit 32 bits.  Forward, both gradients, at sizes that would
otherwise take the large tile.  A bf16 result carries one rounding (2^-8 of the norm allowed)."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("n,h,w,ci,co,r,s,stride,pad", [(100, 130, 3, 64, 64, 3, 3, 3, 1), (90, 116, 2, 72, 136, 3, 3, 2, 1), (64, 130, 5, 64, 136, 5, 5, 1, 0),
                                                        (64, 66, 9, 192, 136, 3, 1, 1, 0), (40, 70, 19, 192, 72, 3, 1, 2, 0)])
def test_one_column(g, n, h, w, ci, co, r, s, stride, pad):
    import torch
    lib, gen = K.lib(), torch.Generator(device="cuda")
    gen.manual_seed(n + h)
    make = lambda *shape: torch.randn(shape, device="cuda", generator=gen).bfloat16()
    ho, wo = (h + 2 * pad - r) // stride + 1, (w + 2 * pad - s) // stride + 1
    assert wo == 1 or s == 1
    x, wt, dy = make(n, h, w, ci), make(co, r, s, ci), make(n, ho, wo, co)
    shape, room = K.ConvShape(n, h, w, ci, co, r, s, stride, pad), 64 * co * r * s * ci * 4
    y, dx, dw = torch.empty_like(dy), torch.empty_like(x), torch.empty_like(wt)
    ws, turned = torch.empty(room, dtype=torch.uint8, device="cuda"), torch.empty(wt.numel(), dtype=torch.bfloat16, device="cuda")
    q = g.stream_ptr()
    g.call(lib.karma_k_conv2d_fwd_bf16, g.ptr(x), g.ptr(wt), g.ptr(y), C.byref(shape), q)
    g.call(lib.karma_k_conv2d_dgrad_bf16, g.ptr(dy), g.ptr(wt), g.ptr(turned), None, g.ptr(dx), C.byref(shape), q)
    g.call(lib.karma_k_conv2d_wgrad_bf16, g.ptr(dy), g.ptr(x), g.ptr(dw), g.ptr(ws), C.c_uint64(room), C.byref(shape), q)
    frame = torch.nn.functional.pad(x.double(), (0, 0, pad, pad, pad, pad))
    grad, out, left = torch.zeros_like(frame), torch.zeros(n * ho * wo, co, dtype=torch.float64, device="cuda"), dy.double().reshape(-1, co)
    rel = lambda got, want: ((got.double() - want).norm() / want.norm()).item()
    for i in range(r):
        for j in range(s):
            at = (slice(None), slice(i, i + (ho - 1) * stride + 1, stride), slice(j, j + (wo - 1) * stride + 1, stride))
            tap, weight = frame[at].reshape(-1, ci), wt[:, i, j].double()
            out += tap @ weight.T.contiguous()
            grad[at] += (left @ weight).reshape(n, ho, wo, ci)
            want = left.T.contiguous() @ tap
            if want.any():
                assert rel(dw[:, i, j], want) <= 2.0 ** -8, (i, j)
            else:       # a tap that meets padding alone
                assert not dw[:, i, j].any(), (i, j)
    assert rel(y.reshape(-1, co), out) <= 2.0 ** -8
    assert rel(dx, grad[:, pad:pad + h, pad:pad + w]) <= 2.0 ** -8
