"""The 64 x 64 tile whose reduction is divided over a workgroup's wavefronts: fewer k-tiles than wavefronts, one and two stages
of them with and without a rest, rows, columns and k one piece past a tile or a piece long, ranges that a second launch adds
up, and all output stages.  Beside it sizes of the 128 x 128 and 256 x 256 tiles whose last tiles hang over the matrix.
A bf16 result carries one rounding (2^-9 per element); fp32 sums add less than that at these lengths."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K

A, B = K.GEMM_A_STRIDED, K.GEMM_B_STRIDED


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def operands(m, n, k, flags, seed=0):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + m + n + k)
    make = lambda *shape: torch.randn(shape, device="cuda", generator=gen).bfloat16()
    a, b = make(m, k), make(n, k)
    return make, a, b, a.t().contiguous() if flags & A else a, b.t().contiguous() if flags & B else b


def close(got, want, scale):
    return ((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * scale).all().item()


SHAPES = [(8, 8, 8), (64, 64, 64), (72, 56, 72), (56, 136, 184), (64, 72, 256), (136, 64, 264), (72, 200, 512), (200, 72, 584), (328, 264, 1096),
          (8, 1032, 2048), (64, 1000, 2048), (1032, 520, 64), (2056, 1032, 136), (1608, 2056, 456), (5000, 2056, 200)]


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("flags", [0, A, B, A | B])
@pytest.mark.parametrize("with_ws", [False, True])
def test_product(g, m, n, k, flags, with_ws):
    import torch
    make, a, b, ad, bd = operands(m, n, k, flags)
    (kernel, _, _, splits), = K.gemm_plan(m, n, k, flags | K.PLAN_TILES, 0, False, 64 * m * n if with_ws else 0)
    assert kernel == {2056: K.PRODUCT_SMALL, 1608: K.PRODUCT_SMALL, 5000: K.PRODUCT_LARGE}.get(m, K.PRODUCT_SLICES)
    assert (splits > 1) == (with_ws and k == 2048)
    bias, res = make(n), make(m, n)
    ws = torch.empty(16 * m * n, device="cuda") if with_ws else None
    c = torch.full((m + 1, n), 7.0, dtype=torch.bfloat16, device="cuda")
    run = lambda out, bi, re, fl: g.call(K.lib().karma_k_gemm_bf16, g.ptr(ad), g.ptr(bd), g.ptr(out), bi, re, m, n, k, fl,
                                         g.ptr(ws) if with_ws else None, C.c_uint64(ws.numel() * 4 if with_ws else 0), g.stream_ptr())
    run(c, g.ptr(bias), g.ptr(res), flags)
    plain, scale = a.double() @ b.double().t(), a.double().abs() @ b.double().abs().t()
    assert close(c[:m], plain + bias.double() + res.double(), scale + 10)
    assert (c[m] == 7.0).all()          # nothing is written past the last row
    acc = make(m, n).float()
    want = plain + acc.double()
    run(acc, None, None, flags | K.GEMM_OUT_F32 | K.GEMM_ACCUMULATE)
    assert ((acc.double() - want).abs() <= 2e-6 * scale + 1e-6).all()


@pytest.mark.parametrize("m,n,k", [(8, 8, 8), (72, 136, 64), (200, 72, 264), (328, 264, 520), (1024, 1024, 256), (1096, 1032, 200)])
def test_gelu_stages_and_column_sums(g, m, n, k):
    import torch
    assert K.gemm_plan(m, n, k, K.PLAN_TILES, K.GEMM_GELU_FWD) == K.gemm_plan(m, n, k, B | K.PLAN_TILES, K.GEMM_GELU_BWD) == [(K.PRODUCT_SLICES, m, n, 1)]
    make, a, b, ad, bd = operands(m, n, k, 0)
    bias, b = make(n), b * 0.1
    c, act = torch.empty(m, n, dtype=torch.bfloat16, device="cuda"), torch.empty(m, n, dtype=torch.bfloat16, device="cuda")
    g.call(K.lib().karma_k_gemm_gelu_bf16, g.ptr(a), g.ptr(b), g.ptr(c), g.ptr(bias), g.ptr(act), m, n, k, 0, K.GEMM_GELU_FWD, g.stream_ptr())
    plain, scale = a.double() @ b.double().t(), a.double().abs() @ b.double().abs().t()
    assert close(c, plain + bias.double(), scale + 10)
    x = c.double().requires_grad_(True)
    y = torch.nn.functional.gelu(x, approximate="tanh")
    assert close(act, y.detach(), torch.full_like(y, 10.0))
    slope, = torch.autograd.grad(y.sum(), x)
    bt, out = b.t().contiguous(), torch.empty_like(c)
    sums, ws = torch.full((n,), 7.0, device="cuda"), torch.empty(((m + 63) // 64 + 1) * n + 4096, device="cuda")
    g.call(K.lib().karma_k_gemm_gelu_bwd_colsum_bf16, g.ptr(a), g.ptr(bt), g.ptr(out), g.ptr(c), g.ptr(sums), g.ptr(ws),
           C.c_uint64(ws.numel() * 4), m, n, k, g.stream_ptr())
    want = plain * slope
    assert close(out, want, scale + 1)
    assert ((sums.double() - want.sum(0)).abs() <= 2.0 ** -8 * want.abs().sum(0) + 1e-3).all()


@pytest.mark.parametrize("m,n,k,kernel", [(72, 136, 64, K.PRODUCT_SLICES), (1608, 2056, 456, K.PRODUCT_SMALL), (4096, 4096, 256, K.PRODUCT_LARGE)])
def test_gelu_derivative_of_huge_values(g, m, n, k, kernel):
    """The derivative is one on the far right and zero on the far left, up to the largest finite value: nothing becomes NaN."""
    import torch
    assert K.gemm_plan(m, n, k, B | K.PLAN_TILES, K.GEMM_GELU_BWD)[0][0] == kernel
    make, a, b, ad, bd = operands(m, n, k, B)
    at = torch.tensor([6.0, 1e4, 1e18, 1.8e19, 1.9e19, 3e19, 5e19, 1e25, 3e38], device="cuda")
    pre = torch.cat([at, -at]).repeat((m * n + 17) // 18)[:m * n].view(m, n).bfloat16()
    out = torch.empty(m, n, dtype=torch.bfloat16, device="cuda")
    g.call(K.lib().karma_k_gemm_gelu_bf16, g.ptr(ad), g.ptr(bd), g.ptr(out), None, g.ptr(pre), m, n, k, B, K.GEMM_GELU_BWD, g.stream_ptr())
    want = torch.where(pre > 0, a.double() @ b.double().t(), 0.0)
    assert close(out, want, a.double().abs() @ b.double().abs().t())      # (at 6 the derivative is one to 1e-6)
