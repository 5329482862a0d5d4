"""The 256 x 256 tile of the bf16 product where its stream of operand tiles crosses from one work item to the next: two
rounds of items and more with two, three and four k-tiles, whole and ragged, every layout and output stage; divided
reductions; weight gradients, whose second operand is gathered, the last range a single k-tile among them; and convolutions
and their input gradients, whose first operand is gathered, with the 256 x 64 tile too.  Each case states through the plan
that it runs on this tile.  Against float64 sums of the same bf16 operands, tile by tile: a bf16
result carries one rounding (2^-9 of an element; 2^-8 of a tile's norm is allowed), fp32 sums less than 1e-5 at these
lengths."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def bf(seed, *shape):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16)


def close_by_tiles(got, want, tol):
    import torch
    pool = lambda t: torch.nn.functional.avg_pool2d(t.square()[None, None], 128, ceil_mode=True)[0, 0]
    return bool((pool(got.double() - want) <= tol * tol * pool(want)).all())


def items(m, n):
    return -(-m // 256) * -(-n // 256)


WHOLE = [(8192, 4096, 128), (8192, 8192, 192), (8192, 4352, 256)]
RAGGED = [(7176, 4104, 128), (7176, 4104, 136), (7184, 4104, 200), (8200, 8192, 192)]


@pytest.mark.parametrize("m,n,k", WHOLE + RAGGED)
@pytest.mark.parametrize("flags", [0, K.GEMM_A_STRIDED, K.GEMM_B_STRIDED, K.GEMM_A_STRIDED | K.GEMM_B_STRIDED])
def test_few_k_tiles_and_several_items(g, m, n, k, flags):
    import torch
    assert K.gemm_plan(m, n, k, flags) == [(K.PRODUCT_LARGE, m, n, 1)] and items(m, n) > 480
    a, b = bf(1, *((k, m) if flags & 1 else (m, k))), bf(2, *((k, n) if flags & 2 else (n, k)))
    want = (a.double().T if flags & 1 else a.double()) @ (b.double() if flags & 2 else b.double().T)
    out = torch.full((m + 1, n), 7.0, device="cuda")
    for f, ref in ((K.GEMM_OUT_F32, want), (K.GEMM_OUT_F32 | K.GEMM_ACCUMULATE, 2 * want)):
        g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), None, None, m, n, k, flags | f, None, C.c_uint64(0), g.stream_ptr())
        assert close_by_tiles(out[:m], ref, 1e-5) and (out[m] == 7).all()
    bias, res = bf(3, n), bf(4, m, n)
    out = torch.full((m + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")
    g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), g.ptr(bias), g.ptr(res), m, n, k, flags, None, C.c_uint64(0),
           g.stream_ptr())
    assert close_by_tiles(out[:m], want + bias.double() + res.double(), 2.0 ** -8) and (out[m] == 7).all()


@pytest.mark.parametrize("m,n,k", [WHOLE[0], RAGGED[1]])
def test_gelu_stages(g, m, n, k):
    import torch
    lib, gelu = K.lib(), lambda x: torch.nn.functional.gelu(x, approximate="tanh")
    assert K.gemm_plan(m, n, k, 0, K.GEMM_GELU_FWD)[0][0] == K.gemm_plan(m, n, k, K.GEMM_B_STRIDED, K.GEMM_GELU_BWD)[0][0] == K.PRODUCT_LARGE
    a, b, bias = bf(5, m, k), bf(6, n, k), bf(7, n)
    pre, act = (torch.empty(m, n, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    g.call(lib.karma_k_gemm_gelu_bf16, g.ptr(a), g.ptr(b), g.ptr(pre), g.ptr(bias), g.ptr(act), m, n, k, 0, K.GEMM_GELU_FWD, g.stream_ptr())
    assert close_by_tiles(pre, a.double() @ b.double().T + bias.double(), 2.0 ** -8)
    assert close_by_tiles(act, gelu(pre.double()), 2.0 ** -8)
    b, aux = bf(8, k, n), bf(9, m, n)
    x = aux.double().requires_grad_()
    gelu(x).sum().backward()
    want = a.double() @ b.double() * x.grad
    sums, ws = torch.empty(n, device="cuda"), torch.empty((m + 63) // 64 * n, device="cuda")
    g.call(lib.karma_k_gemm_gelu_bwd_colsum_bf16, g.ptr(a), g.ptr(b), g.ptr(pre), g.ptr(aux), g.ptr(sums), g.ptr(ws),
           C.c_uint64(ws.numel() * 4), m, n, k, g.stream_ptr())
    assert close_by_tiles(pre, want, 2.0 ** -7)
    assert ((sums.double() - want.sum(0)).abs() <= 1e-4 * want.abs().sum(0)).all()


@pytest.mark.parametrize("m,n,k", [(512, 2048, 35904), (504, 2056, 39928)])
def test_divided_reduction(g, m, n, k):
    import torch
    flags, room = K.GEMM_A_STRIDED | K.GEMM_B_STRIDED, 256 << 20
    (kernel, _, _, splits), = K.gemm_plan(m, n, k, flags, ws_bytes=room)
    assert kernel == K.PRODUCT_LARGE and splits > 1
    a, b, ws = bf(10, k, m), bf(11, k, n), torch.empty(room, dtype=torch.uint8, device="cuda")
    want = a.double().T @ b.double()
    outs = []
    for _ in range(2):
        out = torch.empty(m, n, device="cuda")
        g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), None, None, m, n, k, flags | K.GEMM_OUT_F32, g.ptr(ws),
               C.c_uint64(room), g.stream_ptr())
        outs.append(out)
    assert close_by_tiles(outs[0], want, 1e-5) and torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("n,h,ci,co,r,stride,single", [(42, 65, 72, 200, 3, 1, True), (25, 65, 136, 200, 3, 1, True), (32, 56, 256, 200, 5, 2, False)])
def test_weight_gradient(g, n, h, ci, co, r, stride, single):
    import torch
    pad = r // 2
    ho = (h + 2 * pad - r) // stride + 1
    shape, room = K.ConvShape(n, h, h, ci, co, r, r, stride, pad), 1 << 30
    (kernel, _, _, splits), = K.conv_plan(shape, K.CONV_WGRAD, room)
    pixels = n * ho * ho
    k_tiles, per = -(-pixels // 64), -(-(-(-pixels // splits)) // 64)
    assert kernel == K.PRODUCT_LARGE and splits > 1 and (not single or k_tiles - (splits - 1) * per == 1)
    x, dy = bf(12, n, h, h, ci), bf(13, n, ho, ho, co)
    dw, ws = torch.empty(co, r, r, ci, dtype=torch.bfloat16, device="cuda"), torch.empty(room, dtype=torch.uint8, device="cuda")
    g.call(K.lib().karma_k_conv2d_wgrad_bf16, g.ptr(dy), g.ptr(x), g.ptr(dw), g.ptr(ws), C.c_uint64(room), C.byref(shape), g.stream_ptr())
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    left = dy.reshape(-1, co).double().T.contiguous()
    for i in range(r):
        for j in range(r):
            tap = xp[:, i:i + (ho - 1) * stride + 1:stride, j:j + (ho - 1) * stride + 1:stride].reshape(-1, ci).double()
            assert close_by_tiles(dw[:, i, j], left @ tap, 2.0 ** -8), (i, j)


# several items per workgroup with two to four k-tiles, a gathered first operand, ragged in every direction
@pytest.mark.parametrize("n,h,ci,co,r,stride,pad,kernel", [(35, 55, 16, 136, 3, 1, 0, K.PRODUCT_LARGE), (35, 105, 16, 136, 3, 2, 1, K.PRODUCT_LARGE),
                                                           (13, 87, 16, 200, 3, 1, 1, K.PRODUCT_LARGE), (25, 113, 24, 64, 3, 1, 1, K.PRODUCT_NARROW),
                                                           (25, 224, 8, 64, 7, 2, 3, K.PRODUCT_NARROW)])
def test_gathered_first_operand(g, n, h, ci, co, r, stride, pad, kernel):
    import torch
    lib, ho = K.lib(), (h + 2 * pad - r) // stride + 1
    shape = K.ConvShape(n, h, h, ci, co, r, r, stride, pad)
    assert K.conv_plan(shape, K.CONV_FWD) == [(kernel, n * ho * ho, co, 1)]
    x, w, add = bf(14, n, h, h, ci), bf(15, co, r, r, ci), bf(16, n, ho, ho, co)
    y = torch.full((n + 1, ho, ho, co), 7.0, dtype=torch.bfloat16, device="cuda")
    g.call(lib.karma_k_conv2d_fwd_add_bf16, g.ptr(x), g.ptr(w), g.ptr(add), g.ptr(y), C.byref(shape), g.stream_ptr())
    want = add.double().reshape(-1, co)
    xp = torch.nn.functional.pad(x, (0, 0, pad, pad, pad, pad))
    for i in range(r):
        for j in range(r):
            tap = xp[:, i:i + (ho - 1) * stride + 1:stride, j:j + (ho - 1) * stride + 1:stride].reshape(-1, ci).double()
            want += tap @ w[:, i, j].double().T.contiguous()
    assert close_by_tiles(y[:n].reshape(-1, co), want, 2.0 ** -8) and (y[n] == 7).all()


@pytest.mark.parametrize("n,h,ci,co,r,pad,kernel", [(35, 53, 136, 16, 3, 0, K.PRODUCT_LARGE), (13, 87, 200, 16, 3, 1, K.PRODUCT_LARGE),
                                                    (25, 113, 64, 24, 3, 1, K.PRODUCT_NARROW)])
def test_input_gradient(g, n, h, ci, co, r, pad, kernel):
    import torch
    ho = h + 2 * pad - r + 1
    shape = K.ConvShape(n, h, h, ci, co, r, r, 1, pad)
    assert K.conv_plan(shape, K.CONV_DGRAD) == [(kernel, n * h * h, ci, 1)]
    dy, w, wt = bf(17, n, ho, ho, co), bf(18, co, r, r, ci), torch.empty(r * r * ci * co, dtype=torch.bfloat16, device="cuda")
    dx = torch.full((n + 1, h, h, ci), 7.0, dtype=torch.bfloat16, device="cuda")
    g.call(K.lib().karma_k_conv2d_dgrad_bf16, g.ptr(dy), g.ptr(w), g.ptr(wt), None, g.ptr(dx), C.byref(shape), g.stream_ptr())
    want = torch.zeros(n * h * h, ci, dtype=torch.float64, device="cuda")
    edge = r - 1 - pad
    dyp = torch.nn.functional.pad(dy, (0, 0, edge, edge, edge, edge))
    for i in range(r):
        for j in range(r):
            tap = dyp[:, r - 1 - i:r - 1 - i + h, r - 1 - j:r - 1 - j + h].reshape(-1, co).double()
            want += tap @ w[:, i, j].double()
    assert close_by_tiles(dx[:n].reshape(-1, ci), want, 2.0 ** -8) and (dx[n] == 7).all()
