"""The 128 x 128 tile of the bf16 product and the choice between the tiles, at the sizes where they can go wrong: one
k-tile and fewer, as many as the stages hold and one more, rows and columns one piece past a tile, four stages (few
tiles, long reductions), and stride-2 input gradients by parity (parities without taps or without pixels among them).
A bf16 result carries one rounding (2^-9 per element); fp32 sums add less than that at these lengths."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K
from oracle import cnn, nn
import synth_inputs as si

TOL = 2.0 ** -8


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


@pytest.mark.parametrize("m,n,k", [(8, 8, 8), (128, 128, 64), (136, 120, 128), (120, 264, 136), (256, 128, 264), (128, 256, 320),
                                   (264, 136, 1672), (1000, 520, 2056)])
@pytest.mark.parametrize("flags", [0, K.GEMM_A_STRIDED, K.GEMM_B_STRIDED, K.GEMM_A_STRIDED | K.GEMM_B_STRIDED])
@pytest.mark.parametrize("with_ws", [False, True])
def test_product(g, m, n, k, flags, with_ws):
    import torch
    a, ad = bf(si.normal(1, (m, k)))
    b, bd = bf(si.normal(2, (n, k)))
    bias, biasd = bf(si.normal(3, (n,)))
    res, resd = bf(si.normal(4, (m, n)))
    if flags & K.GEMM_A_STRIDED:
        ad = ad.t().contiguous()
    if flags & K.GEMM_B_STRIDED:
        bd = bd.t().contiguous()
    ws = torch.empty(8 * m * n, dtype=torch.float32, device="cuda") if with_ws else None
    c = torch.full((m + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")
    g.call(K.lib().karma_k_gemm_bf16, g.ptr(ad), g.ptr(bd), g.ptr(c), g.ptr(biasd), g.ptr(resd), m, n, k, flags,
           g.ptr(ws) if with_ws else None, C.c_uint64(ws.numel() * 4 if with_ws else 0), g.stream_ptr())
    ref = a @ b.T + bias + res
    assert g.rel_l2(back(c)[:m], ref) <= TOL
    scale = np.abs(a) @ np.abs(b.T)
    assert np.all(np.abs(back(c)[:m] - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-5 * scale)
    assert np.all(back(c)[m] == 7.0)          # nothing is written past the last row


@pytest.mark.parametrize("n,h,w,ci,co,r,pad", [(1, 1, 1, 8, 8, 1, 0), (2, 5, 4, 24, 136, 1, 0), (2, 6, 7, 16, 8, 2, 0), (3, 9, 8, 136, 40, 3, 1),
                                               (2, 1, 9, 8, 64, 3, 1), (1, 17, 15, 72, 64, 3, 0), (2, 13, 12, 8, 16, 7, 3), (2, 8, 8, 64, 64, 5, 2)])
def test_stride_2_gradient_by_parity(g, n, h, w, ci, co, r, pad):
    import torch
    x, xd = bf(si.normal(5, (n, h, w, ci)))
    wt, wd = bf(si.normal(6, (co, r, r, ci), 0.2))
    ho, wo = cnn.conv_out(h, r, 2, pad), cnn.conv_out(w, r, 2, pad)
    dy, dyd = bf(si.normal(7, (n, ho, wo, co)))
    add, addd = bf(si.normal(8, (n, h, w, ci)))
    dxo, dwo = cnn.conv2d_bwd(x, wt, dy, 2, pad)
    sh = K.binding.ConvShape(n, h, w, ci, co, r, r, 2, pad)
    ws = torch.empty(r * r * ci * co + 8, dtype=torch.bfloat16, device="cuda")
    for with_add in (False, True):
        dx = torch.full((n, h, w, ci), 7.0, dtype=torch.bfloat16, device="cuda")
        g.call(K.lib().karma_k_conv2d_dgrad_bf16, g.ptr(dyd), g.ptr(wd), g.ptr(ws), g.ptr(addd) if with_add else None, g.ptr(dx),
               C.byref(sh), g.stream_ptr())
        ref = dxo + (add if with_add else 0)
        assert g.rel_l2(back(dx), ref) <= TOL or not np.any(ref), with_add
        assert np.all(np.abs(back(dx) - ref) <= 2.0 ** -7 * np.abs(ref) + 1e-4 * max(np.abs(ref).max(), 1e-30)), with_add


# below, at and past a tile of 16 and a wavefront's 16 and 256 k; dx over dy, as a caller may place it
@pytest.mark.parametrize("m,n,k", [(1, 15, 17), (16, 16, 16), (17, 64, 256), (33, 260, 260), (8, 516, 516)])
def test_linear_relu_backward_in_place(g, m, n, k):
    import torch
    x, w, dy, z = (si.normal(20 + i, s).astype(np.float32) for i, s in enumerate([(m, k), (n, k), (m, n), (m, n)]))
    dzo = dy.astype(np.float64) * (z > 0)
    wants = dzo @ w.astype(np.float64), dzo.T @ x.astype(np.float64), dzo.sum(axis=0)
    for in_place in (False, True):
        xd, wd, zd = (g.dev(a, torch.float32) for a in (x, w, z))
        buf = torch.zeros(m * max(n, k), device="cuda")
        buf[:m * n] = g.dev(dy, torch.float32).reshape(-1)
        dx = buf if in_place else torch.empty(m * k, device="cuda")
        dz = torch.empty(m, n, device="cuda"); dw = torch.empty(n, k, device="cuda"); db = torch.empty(n, device="cuda")
        g.call(K.lib().karma_k_linear_relu_bwd_f32, g.ptr(xd), g.ptr(wd), g.ptr(zd), g.ptr(buf), g.ptr(dz), g.ptr(dx), g.ptr(dw),
               g.ptr(db), m, n, k, g.stream_ptr())
        assert np.array_equal(dz.cpu().numpy(), dzo.astype(np.float32))
        for got, want in zip((dx[:m * k].reshape(m, k), dw, db), wants):     # fp32 sums of up to 516 terms
            assert g.rel_l2(got.cpu().numpy(), want) <= 1e-5 or not np.any(want)
