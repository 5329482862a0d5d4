"""Attention forward is no further from 64 bits than its own steps make it: scores and sums in fp32, probabilities rounded to
bf16 against each query's largest score (so that the largest is one, which bf16 holds exactly), the result rounded once."""
import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("b,s,h,d", [(2, 512, 4, 128), (1, 1024, 4, 128), (2, 512, 4, 152), (1, 1024, 4, 152), (8, 128, 4, 152)])
@pytest.mark.parametrize("spread", [1.0, 2.0])
def test_forward_error(g, b, s, h, d, spread):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(s + d)
    qkv = (torch.randn(b, s, 3, h, d, device="cuda", generator=gen) * torch.tensor([spread, 1.0, 1.0], device="cuda")[:, None, None]).bfloat16()
    ctx, lse = torch.empty(b, s, h, d, dtype=torch.bfloat16, device="cuda"), torch.empty(b * h * s, device="cuda")
    g.call(K.lib().karma_k_attention_fwd_bf16, g.ptr(qkv), g.ptr(ctx), g.ptr(lse), b, s, h, d, g.stream_ptr())
    q, k, v = (t.permute(0, 2, 1, 3).double().contiguous() for t in qkv.unbind(2))
    score = q @ k.transpose(-1, -2).contiguous() / d ** 0.5
    score = score.masked_fill(torch.ones(s, s, dtype=torch.bool, device="cuda").triu(1), -float("inf"))
    p = (score - score.amax(-1, keepdim=True)).exp()
    total = p.sum(-1, keepdim=True)
    exact = p @ v / total
    stepped = (p.bfloat16().double() @ v / total).bfloat16().double()
    error = lambda o: ((o - exact).norm() / exact.norm()).item()
    # (the running maximum of the first tiles is not yet the largest score: half a per cent)
    assert error(ctx.permute(0, 2, 1, 3).double()) <= 1.01 * error(stepped)
