"""LayerNorm backward, batch normalisation and the 3 x 3 max pooling's gradient at the sizes where their split of the work
can go wrong: rows and columns one past a workgroup's share, the last row count that is summed without partial results and
the next, rows too wide for one wavefront's registers, more bands of pixels than one round of the finishing sum takes,
odd images, channel groups that are not full, and pooling windows of equal values, of the lowest values and with NaN.
A bf16 result carries one rounding (2^-8 of the norm allowed); fp32 sums of n terms stay within n * 2^-24 of the terms."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
LAST = 512      # rows whose column sums need no partial results

import paper_2008_11421_amd as K
from oracle import cnn, nn
import synth_inputs as si


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def bf(a):
    import torch
    r = nn.bf16_round(np.asarray(a, dtype=np.float32))
    return r.astype(np.float64), torch.from_numpy(r).to(torch.bfloat16).cuda()


def back(t):
    return t.float().cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("rows,h", [(1, 8), (3, 264), (65, 1032), (LAST, 264), (LAST + 1, 264), (LAST + 60, 520), (130, 4256),
                                    (LAST + 2, 3080), (70, 6144)])
@pytest.mark.parametrize("in_place", [False, True])
def test_layernorm_backward(g, rows, h, in_place):
    import torch
    x, xd = bf(si.normal(81, (rows, h), 2.0) + 0.5)
    gam, gd = bf(1.0 + si.normal(82, (h,), 0.2))
    dy, dyd = bf(si.normal(83, (rows, h)))
    add, addd = bf(si.normal(84, (rows, h)))
    _, cache = nn.layernorm_fwd(x, gam, np.zeros(h))
    dxo, dgo, dbo = nn.layernorm_bwd(dy, gam, cache)
    stats = torch.from_numpy(np.stack([x.mean(-1), cache[1].reshape(-1)], 1).astype(np.float32)).cuda()
    dx = dyd if in_place else torch.empty_like(xd)      # the gradient may replace the one it is made from
    dg, db, asum = (torch.full((h,), 7.0, device="cuda") for _ in range(3))
    ws = torch.full(((rows + 63) // 64 * 3 * h,), 7.0, device="cuda")
    g.call(K.lib().karma_k_layernorm_bwd_addsum_bf16, g.ptr(dyd), g.ptr(xd), g.ptr(stats), g.ptr(gd), g.ptr(addd), g.ptr(dx),
           g.ptr(dg), g.ptr(db), g.ptr(asum), g.ptr(ws), C.c_uint64(ws.numel() * 4), rows, h, g.stream_ptr())
    assert g.rel_l2(back(dx), dxo + add) <= 2.0 ** -8
    assert g.elem_ratio(back(dx), dxo + add, 1, 1e-3) <= 1
    xhat = cache[0]
    for got, want, terms in ((dg, dgo, np.abs(dy * xhat).sum(0)), (db, dbo, np.abs(dy).sum(0)), (asum, add.sum(0), np.abs(add).sum(0))):
        # each xhat carries three roundings of its own beside the sum's
        assert (np.abs(got.cpu().numpy() - want.reshape(-1)) <= (rows + 4) * 2.0 ** -24 * terms + 1e-6).all()


@pytest.mark.parametrize("rows,c", [(1, 8), (7, 64), (257, 64), (70000, 24), (140003, 8), (5, 2056)])
def test_batchnorm(g, rows, c):
    import torch
    x, xd = bf(si.normal(85, (rows, c), 1.5) + 0.3)
    gam, gd = bf(1.0 + si.normal(86, (c,), 0.2))
    bet, bd = bf(si.normal(87, (c,), 0.2))
    dy, dyd = bf(si.normal(88, (rows, c)))
    lib = K.lib()
    size = lib.karma_k_batchnorm_ws_bytes
    size.restype = C.c_uint64
    ws = torch.full((int(size(C.c_uint32(rows), C.c_uint32(c))),), 255, dtype=torch.uint8, device="cuda")
    y, dx = torch.empty_like(xd), torch.empty_like(xd)
    stats, dg, db = torch.empty(2 * c, device="cuda"), torch.empty(c, device="cuda"), torch.empty(c, device="cuda")
    g.call(lib.karma_k_batchnorm_fwd_bf16, g.ptr(xd), g.ptr(gd), g.ptr(bd), None, g.ptr(y), g.ptr(stats), g.ptr(ws), rows, c, 0,
           g.stream_ptr())
    mean, var = x.mean(0), x.var(0)
    rstd = 1.0 / np.sqrt(var + 1e-5)
    xhat = (x - mean) * rstd
    assert np.allclose(stats[:c].cpu().numpy(), mean, rtol=0, atol=rows * 2.0 ** -24 * 8 + 1e-6)
    want = xhat * gam + bet
    assert np.abs(back(y) - want).max() <= 2.0 ** -8 * np.abs(want).max()
    g.call(lib.karma_k_batchnorm_bwd_bf16, g.ptr(dyd), g.ptr(xd), g.ptr(stats), g.ptr(gd), g.ptr(bd), 0, g.ptr(dx), g.ptr(dg),
           g.ptr(db), g.ptr(ws), rows, c, g.stream_ptr())
    # sums in blocks of a few hundred: far fewer additions in a row than rows, 2^-20 of the terms covers them
    assert (np.abs(db.cpu().numpy() - dy.sum(0)) <= 2.0 ** -20 * np.abs(dy).sum(0) + 1e-6).all()
    if rows > 7:       # with a handful of rows the variance itself is a difference of roundings
        assert (np.abs(dg.cpu().numpy() - (dy * xhat).sum(0)) <= 2.0 ** -18 * np.abs(dy * xhat).sum(0) + 1e-4).all()
        ref = gam * rstd * (dy - dy.mean(0) - xhat * (dy * xhat).mean(0))
        assert g.rel_l2(back(dx), ref) <= 2.0 ** -8


@pytest.mark.parametrize("n,h,w,c", [(1, 1, 1, 8), (2, 1, 5, 24), (1, 2, 2, 64), (2, 15, 17, 40), (1, 16, 33, 72), (3, 34, 18, 32),
                                     (1, 112, 112, 64)])
def test_maxpool_gradient(g, n, h, w, c):
    """Against a direct evaluation of the rule: dy goes to the first largest element of its window, and to none where the
    window holds a NaN beside other elements."""
    import torch
    x = nn.bf16_round(np.round(si.normal(89, (n, h, w, c), 1.5)).astype(np.float32))      # many equal values
    x.reshape(-1)[::7] = 0.0
    x.reshape(-1)[::11] = -0.0
    x[:, h // 2:, :w // 2, ::3] = -np.inf
    x[:, ::6, ::5, 1::8] = np.nan
    ho, wo = (h - 1) // 2 + 1, (w - 1) // 2 + 1
    dy = nn.bf16_round(si.normal(90, (n, ho, wo, c)).astype(np.float32))
    xd, dyd = (torch.from_numpy(a).to(torch.bfloat16).cuda() for a in (x, dy))
    dx = torch.full_like(xd, 7.0)
    g.call(K.lib().karma_k_maxpool_bwd_bf16, g.ptr(xd), g.ptr(dyd), g.ptr(dx), n, h, w, c, g.stream_ptr())
    ref = np.zeros(x.shape, np.float32)
    for i in range(ho):
        for j in range(wo):
            at = [(r, s) for r in range(2 * i - 1, 2 * i + 2) for s in range(2 * j - 1, 2 * j + 2) if 0 <= r < h and 0 <= s < w]
            v = np.stack([x[:, r, s] for r, s in at])
            first = np.where(np.isnan(v).any(0) & (len(at) > 1), -1, np.argmax(np.where(np.isnan(v), -np.inf, v), axis=0))
            for k, (r, s) in enumerate(at):
                ref[:, r, s] += np.where(first == k, dy[:, i, j], 0)
    assert np.array_equal(dx.float().cpu().numpy(), nn.bf16_round(ref))
