"""Products whose operands allow no 16-byte pieces (row counts of strided operands that are no multiples of 8, operands that
start between 16-byte boundaries): the register-staged kernel with its 128 x 128 and its 256 x 256 tile, every layout and
output stage, with and without divided reductions.  Against float64 products of the same bf16 operands; a bf16 result
carries one rounding (2^-9 of an element; 2^-8 of the norm is allowed), fp32 results sums of K terms."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def operand(rows, k, strided, off, seed):
    """(rows x k values, device tensor that starts 2 * off bytes after a 16-byte boundary)"""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    room = torch.randn(rows * k + 8, device="cuda", generator=gen).to(torch.bfloat16)[off:off + rows * k]
    return room, (room.reshape(k, rows).T if strided else room.reshape(rows, k)).double()


def close(got, want, tol):
    assert ((got.double() - want).norm() / want.norm()).item() <= tol
    for r in (slice(0, 128), slice(-132, None)):        # block by block, so that a wrong edge cannot hide in the norm
        for c in (slice(0, 128), slice(-132, None)):
            assert ((got.double() - want)[r, c].norm() / want[r, c].norm()).item() <= tol


# (sizes, first element): small tile and large tile, rows that are no octets, two rounds and a ragged third, whole tiles
SIZES = [(132, 236, 72, 0), (264, 520, 136, 4), (700, 1820, 1000, 0), (3844, 4092, 1032, 0), (4096, 4096, 1024, 4), (4100, 8196, 520, 0)]


@pytest.mark.parametrize("m,n,k,off", SIZES)
@pytest.mark.parametrize("flags", [0, K.GEMM_A_STRIDED, K.GEMM_B_STRIDED, K.GEMM_A_STRIDED | K.GEMM_B_STRIDED])
@pytest.mark.parametrize("with_ws", [False, True])
def test_layouts(g, m, n, k, off, flags, with_ws):
    import torch
    off = off or (4 if flags != 3 else 0)               # (only strided rows of fours need no shifted start)
    a, av = operand(m, k, flags & 1, off, 1)
    b, bv = operand(n, k, flags & 2, off, 2)
    bias, bias_v = operand(n, 1, False, 0, 3)
    res, res_v = operand(m, n, False, 0, 4)
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda") if with_ws else None
    guard = torch.full((m + 2, n), 7.0, dtype=torch.bfloat16, device="cuda")
    out = guard[1:-1]
    g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), g.ptr(bias), g.ptr(res), m, n, k, flags,
           g.ptr(ws) if with_ws else None, C.c_uint64(64 << 20 if with_ws else 0), g.stream_ptr())
    close(out, av @ bv.T + bias_v.T + res_v, 2.0 ** -8)
    assert (guard[0] == 7).all() and (guard[-1] == 7).all()


@pytest.mark.parametrize("m,n,k", [(65537, 8, 8), (65664, 128, 64), (140001, 37, 24)])
def test_one_k_tile_and_one_column_of_tiles(g, m, n, k):
    import torch
    assert K.gemm_plan(m, n, k) == [(K.PRODUCT_STAGED_SMALL, m, n, 1)]
    a, av = operand(m, k, False, 0, 9)
    b, bv = operand(n, k, False, 0, 10)
    bias, bias_v = operand(n, 1, False, 0, 11)
    res, res_v = operand(m, n, False, 0, 12)
    guard = torch.full((m + 2, n), 7.0, dtype=torch.bfloat16, device="cuda")
    out = guard[1:-1]
    g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), g.ptr(bias), g.ptr(res), m, n, k, 0, None, C.c_uint64(0),
           g.stream_ptr())
    want = av @ bv.T + bias_v.T + res_v
    assert ((out.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all()
    assert (guard[0] == 7).all() and (guard[-1] == 7).all()


@pytest.mark.parametrize("m,n,k", [(264, 520, 136), (3844, 4092, 1032)])
def test_output_stages(g, m, n, k):
    import torch
    a, av = operand(m, k, False, 4, 5)
    b, bv = operand(n, k, False, 4, 6)
    want = av @ bv.T
    out = torch.full((m, n), 3.0, device="cuda")
    for flags, ref in ((K.GEMM_OUT_F32, want), (K.GEMM_OUT_F32 | K.GEMM_ACCUMULATE, 2 * want)):
        g.call(K.lib().karma_k_gemm_bf16, g.ptr(a), g.ptr(b), g.ptr(out), None, None, m, n, k, flags, None, C.c_uint64(0), g.stream_ptr())
        close(out, ref, 1e-5)
    gelu = lambda x: torch.nn.functional.gelu(x, approximate="tanh")
    pre, act = (torch.empty(m, n, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    fn = K.lib().karma_k_gemm_gelu_bf16
    g.call(fn, g.ptr(a), g.ptr(b), g.ptr(pre), None, g.ptr(act), m, n, k, 0, K.GEMM_GELU_FWD, g.stream_ptr())
    close(pre, want, 2.0 ** -8)
    close(act, gelu(pre.double()), 2.0 ** -8)
    b, bv = operand(n, k, True, 4, 7)
    aux, aux_v = operand(m, n, False, 0, 8)
    x = aux_v.clone().requires_grad_()
    gelu(x).sum().backward()
    g.call(fn, g.ptr(a), g.ptr(b), g.ptr(pre), None, g.ptr(aux), m, n, k, K.GEMM_B_STRIDED, K.GEMM_GELU_BWD, g.stream_ptr())
    close(pre, av @ bv.T * x.grad, 2.0 ** -7)
