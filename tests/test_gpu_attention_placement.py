"""Attention backward with results over inputs that it has read by then: the gradients over the forward's output, and the
column sums' workspace over any input.  Against the same call with buffers of their own: what the two add up in another
order (delta, over the head dimension in fp32; the column sums, from the rounded gradients) moves a result by one rounding
here and there."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def problem(g, b, s, h, d):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(b + s + h + d)
    make = lambda *shape: torch.randn(shape, device="cuda", generator=gen).bfloat16()
    qkv, dctx = make(b * s, 3 * h * d), make(b * s, h * d)
    ctx, lse = torch.empty_like(dctx), torch.empty(b * h * s, device="cuda")
    g.call(K.lib().karma_k_attention_fwd_bf16, g.ptr(qkv), g.ptr(ctx), g.ptr(lse), b, s, h, d, g.stream_ptr())
    return qkv, dctx, ctx, lse, torch.empty_like(lse), torch.empty_like(qkv)


def rel(got, want):
    return ((got.double() - want.double()).norm() / want.double().norm()).item()


@pytest.mark.parametrize("b,s,h,d", [(2, 256, 3, 64), (2, 384, 3, 128), (1, 512, 2, 152), (3, 128, 5, 152)])
@pytest.mark.parametrize("third", [0, 1, 2])
def test_gradients_over_the_output(g, b, s, h, d, third):
    import torch
    qkv, dctx, ctx, lse, delta, want = problem(g, b, s, h, d)
    fn = K.lib().karma_k_attention_bwd_bf16
    g.call(fn, g.ptr(qkv), g.ptr(ctx), g.ptr(dctx), g.ptr(lse), g.ptr(delta), g.ptr(want), b, s, h, d, g.stream_ptr())
    got = torch.empty_like(want)
    inside = got.reshape(3, -1)[third].view(b * s, h * d)
    inside.copy_(ctx)
    g.call(fn, g.ptr(qkv), g.ptr(inside), g.ptr(dctx), g.ptr(lse), g.ptr(delta), g.ptr(got), b, s, h, d, g.stream_ptr())
    for part in range(3):      # the gradients of q, k and v
        cols = slice(part * h * d, (part + 1) * h * d)
        assert rel(got[:, cols], want[:, cols]) <= 2.0 ** -9, part


@pytest.mark.parametrize("b,s,h,d", [(2, 256, 3, 64), (2, 384, 3, 128), (1, 512, 2, 152)])
@pytest.mark.parametrize("over", ["qkv", "ctx", "dctx"])
def test_column_sums_workspace_over_inputs(g, b, s, h, d, over):
    import torch
    qkv, dctx, ctx, lse, delta, dqkv = problem(g, b, s, h, d)
    nbytes = b * s // 32 * 3 * h * d * 4
    ws, sums, want = torch.empty(nbytes // 4, device="cuda"), torch.empty(3 * h * d, device="cuda"), torch.empty_like(dqkv)
    run = lambda ws, out: g.call(K.lib().karma_k_attention_bwd_colsum_bf16, g.ptr(qkv), g.ptr(ctx), g.ptr(dctx), g.ptr(lse), g.ptr(delta),
                                 g.ptr(out), g.ptr(sums), g.ptr(ws), C.c_uint64(nbytes), b, s, h, d, g.stream_ptr())
    run(ws, want)
    first = sums.clone()
    size = want.double().abs().sum(0)
    assert ((first.double() - want.double().sum(0)).abs() <= 2.0 ** -8 * size + 1e-6).all()
    run(dict(qkv=qkv, ctx=ctx, dctx=dctx)[over], dqkv)
    assert torch.equal(dqkv, want)
    assert ((sums.double() - want.double().sum(0)).abs() <= 1e-5 * size + 1e-6).all()
