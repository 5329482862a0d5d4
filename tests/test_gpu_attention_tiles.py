"""The attention kernels at the head dimensions whose tiles are two whole panels of 64 columns (128) or end in a part of one
(152): bias gradients of all three thirds, few workgroups and more than one per compute unit, one query tile and several,
and a neighbouring head full of huge values, which a padded column must not take in.
Tolerance: three chained bf16 roundings (probabilities, their gradients, results; delta from the stored context) leave
about 1 % of a head's gradient, as for head dimension 64; a bias gradient is a sum of those."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K
from oracle import nn
import synth_inputs as si

TOL = 1e-2


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("B,S,H,D", [(1, 1152, 2, 64), (1, 1024, 1, 152), (1, 640, 2, 128), (1, 128, 1, 128), (4, 512, 17, 128), (1, 128, 1, 152), (1, 384, 3, 152), (3, 512, 22, 152)])
@pytest.mark.parametrize("huge_head", [False, True])
def test_forward_backward_and_bias_gradient(g, B, S, H, D, huge_head):
    import torch
    h = H * D
    x = si.normal(71, (B, S, 3 * h), 1.2)
    dy = si.normal(72, (B, S, h))
    if huge_head:      # the last head's inputs are 2^40 times larger: its products stay finite, and its neighbour's do not see them
        x.reshape(B, S, 3, H, D)[:, :, 2, H - 1] *= 2.0 ** 40
    x, dy = nn.bf16_round(x.astype(np.float32)), nn.bf16_round(dy.astype(np.float32))
    to = lambda a: torch.from_numpy(a).to(torch.bfloat16).cuda()
    back = lambda t: t.float().cpu().numpy().astype(np.float64)
    qkv, dctx, lib = to(x), to(dy), K.lib()
    ctx = torch.empty(B, S, h, dtype=torch.bfloat16, device="cuda")
    lse, delta = torch.empty(B, H, S, device="cuda"), torch.empty(B, H, S, device="cuda")
    dqkv, sums = torch.empty_like(qkv), torch.empty(3 * h, device="cuda")
    ws = torch.empty(B * S // 32 * 3 * h, device="cuda")
    g.call(lib.karma_k_attention_fwd_bf16, g.ptr(qkv), g.ptr(ctx), g.ptr(lse), B, S, H, D, g.stream_ptr())
    g.call(lib.karma_k_attention_bwd_colsum_bf16, g.ptr(qkv), g.ptr(ctx), g.ptr(dctx), g.ptr(lse), g.ptr(delta), g.ptr(dqkv),
           g.ptr(sums), g.ptr(ws), C.c_uint64(ws.numel() * 4), B, S, H, D, g.stream_ptr())
    x64 = x.astype(np.float64)
    ref, probs = nn.mha_fwd(x64, H)
    grad = nn.mha_bwd(x64, H, probs, dy.astype(np.float64))
    got, grad, want = back(dqkv).reshape(B, S, 3, H, D), grad.reshape(B, S, 3, H, D), ref.reshape(B, S, H, D)
    bias = sums.cpu().numpy().reshape(3, H, D)
    for j in range(H):
        assert g.rel_l2(back(ctx).reshape(B, S, H, D)[:, :, j], want[:, :, j]) <= TOL, j
        assert g.rel_l2(bias[2, j], grad[:, :, 2, j].sum((0, 1))) <= TOL, j
        for t in range(3):
            if huge_head and j == H - 1 and t < 2:
                continue      # differences of numbers 2^40 large: nothing of them is left to compare
            assert g.rel_l2(got[:, :, t, j], grad[:, :, t, j]) <= TOL, (j, t)
    # key and query biases: sums that nearly cancel (a key bias shifts every score of a query alike), so against the
    # terms: each carries the 1 % above, and their errors add at most like the terms' sizes
    for t in range(2):
        terms = np.abs(grad[:, :, t, :H - 1 if huge_head else H]).sum((0, 1))
        err = np.abs(bias[t] - grad[:, :, t].sum((0, 1)))[:H - 1 if huge_head else H]
        assert (err <= TOL * terms + 1e-6).all(), (t, (err / (terms + 1e-30)).max())
