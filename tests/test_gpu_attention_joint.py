"""Attention where the chip is far from full: two groups of wavefronts on a workgroup's key tiles forward, both backward passes
in one launch (with one group of wavefronts or two), and (batch, head) pairs that are no multiple of eight.  At the edges of
the rules that choose them, on a chip of 256 compute units: tiles * heads * batch of 128, 192, 256 and 512, sequences of 256,
512 and 640.  Against float64.
Tolerance as for the other attention tests: three chained bf16 roundings leave about 1 % of a head's gradient."""
import ctypes as C
import math

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K

TOL = 1e-2


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


SHAPES = [(1, 128, 1, 64), (5, 256, 3, 64), (1, 384, 3, 64), (2, 512, 16, 64), (3, 512, 11, 64), (3, 640, 12, 64), (4, 1024, 8, 64), (4, 1024, 16, 64),
          (5, 896, 15, 64), (2, 384, 5, 128), (1, 512, 9, 128), (3, 640, 12, 128), (4, 512, 12, 128), (1, 256, 3, 152), (3, 640, 11, 152),
          (4, 512, 16, 152),
          (3, 1408, 17, 64), (1, 1408, 35, 152)]        # (the last two: all pairs dealt tile by tile)


def reference(qkv, dctx, b, s, h, d):
    import torch
    x = qkv.double().view(b, s, 3, h, d).permute(2, 0, 3, 1, 4).contiguous()
    q, k, v = x[0], x[1], x[2]
    do = dctx.double().view(b, s, h, d).permute(0, 2, 1, 3).contiguous()
    sc = torch.matmul(q, k.transpose(-1, -2).contiguous()) / d ** 0.5
    sc = sc.masked_fill(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    p = torch.softmax(sc, -1)
    o = torch.matmul(p, v)
    dp = torch.matmul(do, v.transpose(-1, -2).contiguous())
    ds = p * (dp - (dp * p).sum(-1, keepdim=True)) / d ** 0.5
    pt, dst = p.transpose(-1, -2).contiguous(), ds.transpose(-1, -2).contiguous()
    return o, torch.stack([torch.matmul(ds, k), torch.matmul(dst, q), torch.matmul(pt, do)])


@pytest.mark.parametrize("b,s,h,d", SHAPES)
def test_against_float64(g, b, s, h, d):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(s + h)
    make = lambda *shape: torch.randn(shape, device="cuda", generator=gen).bfloat16()
    qkv, dctx, lib = make(b, s, 3 * h * d), make(b, s, h * d), K.lib()
    ctx, lse, delta = torch.empty_like(dctx), torch.empty(b * h * s, device="cuda"), torch.empty(b * h * s, device="cuda")
    dqkv, sums, ws = torch.empty_like(qkv), torch.empty(3 * h * d, device="cuda"), torch.empty(b * s // 32 * 3 * h * d, device="cuda")
    g.call(lib.karma_k_attention_fwd_bf16, g.ptr(qkv), g.ptr(ctx), g.ptr(lse), b, s, h, d, g.stream_ptr())
    g.call(lib.karma_k_attention_bwd_colsum_bf16, g.ptr(qkv), g.ptr(ctx), g.ptr(dctx), g.ptr(lse), g.ptr(delta), g.ptr(dqkv), g.ptr(sums),
           g.ptr(ws), C.c_uint64(ws.numel() * 4), b, s, h, d, g.stream_ptr())
    o, grad = reference(qkv, dctx, b, s, h, d)
    got_o = ctx.double().view(b, s, h, d).permute(0, 2, 1, 3)
    got = dqkv.double().view(b, s, 3, h, d).permute(2, 0, 3, 1, 4)
    per = lambda x, y: ((x - y).pow(2).sum((-1, -2)) / y.pow(2).sum((-1, -2))).sqrt().max().item()      # worst (batch, head)
    assert per(got_o, o) <= TOL
    for t in range(3):
        assert per(got[t], grad[t]) <= TOL, t
    got_delta = delta.view(b, h, s).double()
    want_delta = (dctx.double() * ctx.double()).view(b, s, h, d).sum(-1).permute(0, 2, 1)
    assert (got_delta - want_delta).abs().max().item() <= 1e-4 * d ** 0.5
    # the bias gradients: sums over all tokens of terms that each carry the error above
    terms = grad.abs().sum((1, 3))
    err = (sums.double().view(3, h, d) - grad.sum((1, 3))).abs()
    assert (err <= TOL * terms + 1e-6).all()


@pytest.mark.parametrize("s", [512, 640])
def test_scores_of_minus_infinity(g, s):
    """Keys whose every score is minus infinity, a whole tile of them among others: nothing of them is seen."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(s)
    qkv = torch.randn((1, s, 3, 2, 64), device="cuda", generator=gen).bfloat16()
    qkv[:, :, 0, :, 0] = 1.0
    out = []
    for low in (-1e30, float("-inf")):
        x = qkv.clone()
        x[:, 64:128, 1, :, 0] = low
        x[:, 64:128, 0] = torch.randn((1, 64, 2, 64), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1)).bfloat16()
        x[:, 64:128, 0, :, 0] = 1.0
        ctx, lse = torch.empty((1, s, 128), device="cuda", dtype=torch.bfloat16), torch.empty(2 * s, device="cuda")
        g.call(K.lib().karma_k_attention_fwd_bf16, g.ptr(x), g.ptr(ctx), g.ptr(lse), 1, s, 2, 64, g.stream_ptr())
        out.append((ctx.clone(), lse.clone()))
    assert torch.isfinite(out[1][0].float()).all() and torch.isfinite(out[1][1]).all()
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("s,d,first", [(256, 152, 32), (384, 152, 32), (512, 64, 64), (640, 64, 64), (512, 128, 64), (768, 128, 64)])
def test_minus_infinity_for_some_queries(g, s, d, first):
    """Finite values whose scores overflow to minus infinity for every other query, on the second group's first tile (and, for
    one head, on the first group's as well): what a wavefront rescales for its other queries is not to touch these."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(s + d)
    qkv = torch.randn((1, s, 3, 2, d), device="cuda", generator=gen).bfloat16()
    qkv[:, :, 0, :, 0] = 2.0 * (torch.arange(s, device="cuda") % 2)[None, :, None]
    qkv[:, first:2 * first, 1, :, 0] = -3e38
    qkv[:, 1:first, 1, 1, 0] = -3e38
    ctx, lse = torch.empty((1, s, 2 * d), device="cuda", dtype=torch.bfloat16), torch.empty((2, s), device="cuda")
    g.call(K.lib().karma_k_attention_fwd_bf16, g.ptr(qkv), g.ptr(ctx), g.ptr(lse), 1, s, 2, d, g.stream_ptr())
    x = qkv.double().permute(2, 0, 3, 1, 4).contiguous()[:, 0]
    sc = torch.matmul(x[0], x[1].transpose(-1, -2).contiguous()) / d ** 0.5
    sc = sc.masked_fill(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    want = torch.matmul(torch.softmax(sc, -1), x[2])
    got = ctx.double().view(s, 2, d).permute(1, 0, 2)
    assert torch.isfinite(got).all() and torch.isfinite(lse).all()
    assert ((got - want).pow(2).sum((-1, -2)) / want.pow(2).sum((-1, -2))).sqrt().max().item() <= TOL
    assert (lse.double() - torch.logsumexp(sc, -1) / math.log(2)).abs().max().item() <= 1e-3       # fp32 sums of exact products
