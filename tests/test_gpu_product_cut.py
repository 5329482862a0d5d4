"""Products cut in two, whole rounds of large tiles and a rest: along columns and along rows, every layout, with and without
room for the rest's ranges of the reduction, with each of the output stages.  Against float64 products of the same bf16
operands; a bf16 result carries one rounding (2^-9 of an element; 2^-8 of the norm is allowed), fp32 results sums of K terms."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def operands(m, n, k, a_strided, b_strided):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + 3 * n + 7 * k)
    make = lambda *shape: torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16)
    a, b = make(*((k, m) if a_strided else (m, k))), make(*((k, n) if b_strided else (n, k)))
    want = (a.double().T if a_strided else a.double()) @ (b.double() if b_strided else b.double().T)
    return make, a, b, want


def close(got, want, tol):
    assert ((got.double() - want).norm() / want.norm()).item() <= tol
    # block by block, so that a wrong edge cannot hide in the norm
    for r in (slice(0, 256), slice(-136, None)):
        for c in (slice(0, 256), slice(-136, None)):
            assert ((got.double() - want)[r, c].norm() / want[r, c].norm()).item() <= tol


# 16 x 17 and 17 x 16 large tiles (cut along columns, along rows), 17 x 17, and one and a half rounds of whole tiles
SIZES = [(4096, 4136, 2048), (4104, 4096, 2056), (4160, 4128, 2048), (4096, 6144, 2048)]


@pytest.mark.parametrize("m,n,k", SIZES)
@pytest.mark.parametrize("flags", [0, K.GEMM_A_STRIDED, K.GEMM_B_STRIDED, K.GEMM_A_STRIDED | K.GEMM_B_STRIDED])
def test_layouts(g, m, n, k, flags):
    import torch
    make, a, b, want = operands(m, n, k, flags & K.GEMM_A_STRIDED, flags & K.GEMM_B_STRIDED)
    bias, res, ws = make(n), make(m, n), torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    outs = []
    for w in (None, ws):
        guard = torch.full((m + 2, n), 7.0, dtype=torch.bfloat16, device="cuda")
        out = guard[1:-1]
        g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), g.ptr(bias), g.ptr(res), m, n, k, flags,
               g.ptr(w) if w is not None else None, C.c_uint64(w.numel() if w is not None else 0), g.stream_ptr())
        close(out, want + bias.double() + res.double(), 2.0 ** -8)
        assert (guard[0] == 7).all() and (guard[-1] == 7).all()
        outs.append(out)
    close(outs[1], outs[0].double(), 2.0 ** -8)


@pytest.mark.parametrize("m,n,k", SIZES[:2])
def test_fp32_and_accumulating_results(g, m, n, k):
    import torch
    _, a, b, want = operands(m, n, k, False, False)
    out = torch.full((m, n), 3.0, device="cuda")
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), None, None, m, n, k, K.GEMM_OUT_F32, g.ptr(ws),
           C.c_uint64(ws.numel()), g.stream_ptr())
    close(out, want, 1e-5)
    g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), None, None, m, n, k,
           K.GEMM_OUT_F32 | K.GEMM_ACCUMULATE, g.ptr(ws), C.c_uint64(ws.numel()), g.stream_ptr())
    close(out, 2 * want, 1e-5)


@pytest.mark.parametrize("m,n,k", SIZES[:3])
def test_gelu_stages(g, m, n, k):
    import torch
    make, a, b, want = operands(m, n, k, False, False)
    bias, pre, act = make(n), torch.empty(m, n, dtype=torch.bfloat16, device="cuda"), torch.empty(m, n, dtype=torch.bfloat16, device="cuda")
    gelu = lambda x: torch.nn.functional.gelu(x, approximate="tanh")
    fn = K.lib().karma_k_gemm_gelu_bf16
    g.call(fn, g.ptr(a), g.ptr(b), g.ptr(pre), g.ptr(bias), g.ptr(act), m, n, k, 0, K.GEMM_GELU_FWD, g.stream_ptr())
    close(pre, want + bias.double(), 2.0 ** -8)
    close(act, gelu(pre.double()), 2.0 ** -8)
    _, a, b, want = operands(m, n, k, False, True)
    x = make(m, n).double().requires_grad_()
    gelu(x).sum().backward()
    out, aux = torch.empty_like(pre), x.detach().to(torch.bfloat16)
    g.call(fn, g.ptr(a), g.ptr(b), g.ptr(out), None, g.ptr(aux), m, n, k, K.GEMM_B_STRIDED, K.GEMM_GELU_BWD, g.stream_ptr())
    close(out, want * x.grad, 2.0 ** -7)
