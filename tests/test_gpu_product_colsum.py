"""The feed-forward gradient with the column sums of its result: the workspace that karma.h asks for, ceil(m / 64) rows of n
floats, and not a float more, at row counts around the tiles' edges, on both tiles.
Against float64 products of the same bf16 operands: a bf16 result carries its own rounding and that of GELU'; the sums are
fp32 sums of m terms, of rounded ones where they are taken from the stored result."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("m", [1, 63, 64, 65, 127, 128, 129, 192, 193, 256, 257, 320])
@pytest.mark.parametrize("n,k", [(8, 8), (136, 72), (520, 40)])
def test_workspace_is_what_the_header_says(g, m, n, k):
    run(g, m, n, k)


@pytest.mark.parametrize("m,n,k", [(8192, 4096, 128), (7176, 4104, 136), (4096, 4104, 2048)])
def test_large_tile(g, m, n, k):
    assert K.gemm_plan(m, n, k, K.GEMM_B_STRIDED, K.GEMM_GELU_BWD)[0][0] == K.PRODUCT_LARGE
    run(g, m, n, k)


def run(g, m, n, k):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(m + n + k)
    a, b, aux = (torch.randn(s, device="cuda", generator=gen).bfloat16() for s in ((m, k), (k, n), (m, n)))
    floats = (m + 63) // 64 * n
    ws = torch.full((floats + 4096,), 7.0, device="cuda")
    out, sums = torch.empty(m, n, dtype=torch.bfloat16, device="cuda"), torch.empty(n, device="cuda")
    args = lambda nbytes: (g.ptr(a), g.ptr(b), g.ptr(out), g.ptr(aux), g.ptr(sums), g.ptr(ws), C.c_uint64(nbytes), m, n, k, g.stream_ptr())
    fn = K.lib().karma_k_gemm_gelu_bwd_colsum_bf16
    assert fn(*args(floats * 4 - 4)) == K.E_OOM
    g.call(fn, *args(floats * 4))
    assert (ws[floats:] == 7).all()
    x = aux.double().requires_grad_()
    torch.nn.functional.gelu(x, approximate="tanh").sum().backward()
    want = a.double() @ b.double() * x.grad
    assert ((out.double() - want).norm() / want.norm()).item() <= 2.0 ** -7
    assert ((sums.double() - want.sum(0)).abs() <= (2.0 ** -8 + 1e-5) * want.abs().sum(0) + 1e-6).all()
