"""Both gradients of a linear layer in one call, in one launch of the 64 x 64 tile where the plan says so: rows, widths and k one
piece past a tile or a piece long, odd numbers of rows, one and two stages of k-tiles, the GELU stage with its column sums, fp32
results added to what is there; and sizes that are two launches.  Against float64: a bf16 result carries one rounding (2^-9 per
element), fp32 sums less than 1e-5 at these lengths."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K

TOGETHER = [(1, 8, 8), (65, 72, 56), (200, 256, 72), (256, 264, 248), (327, 264, 1032), (1000, 136, 328), (1027, 520, 256), (2049, 264, 200),
            (3111, 512, 128), (2048, 1024, 1024)]
APART = [(3840, 3040, 760), (4160, 256, 256)]


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def close(got, want, scale):
    return ((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5 * scale).all().item()


@pytest.mark.parametrize("rows,n,k", TOGETHER + APART)
@pytest.mark.parametrize("gelu", [False, True])
@pytest.mark.parametrize("added", [False, True])
def test_both_gradients(g, rows, n, k, gelu, added):
    import torch
    flags, room = (K.GEMM_OUT_F32 | K.GEMM_ACCUMULATE if added else 0), 8 * n * k * 4
    if not gelu:
        assert K.linear_bwd_together(rows, n, k, gelu, flags, room) == ((rows, n, k) in TOGETHER)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + n + k)
    make = lambda *shape: torch.randn(shape, device="cuda", generator=gen).bfloat16()
    dy, w, x, aux = make(rows, n), make(n, k), make(rows, k), make(rows, k)
    dx = torch.full((rows + 1, k), 7.0, dtype=torch.bfloat16, device="cuda")
    dw = torch.full((n + 1, k), 7.0, dtype=torch.float32 if added else torch.bfloat16, device="cuda")
    sums, sum_room = torch.full((k,), 7.0, device="cuda"), ((rows + 63) // 64 * k * 4 + 255) // 256 * 256 if gelu else 0
    ws = torch.empty(sum_room + room, dtype=torch.uint8, device="cuda")
    g.call(K.lib().karma_k_linear_bwd_bf16, g.ptr(dy), g.ptr(w), g.ptr(x), g.ptr(dx), g.ptr(dw), g.ptr(aux) if gelu else None,
           g.ptr(sums) if gelu else None, g.ptr(ws), C.c_uint64(ws.numel()), rows, n, k, flags, g.stream_ptr())
    want, scale = dy.double() @ w.double(), dy.double().abs() @ w.double().abs()
    if gelu:
        at = aux.double().requires_grad_(True)
        slope, = torch.autograd.grad(torch.nn.functional.gelu(at, approximate="tanh").sum(), at)
        want, scale = want * slope, scale * slope.abs().clamp(min=1.0)
        assert ((sums.double() - want.sum(0)).abs() <= 2.0 ** -8 * want.abs().sum(0) + 1e-3).all()
    assert close(dx[:rows], want, scale + 1e-3) and (dx[rows] == 7).all()
    want, scale = dy.double().T @ x.double(), dy.double().abs().T @ x.double().abs()
    assert (dw[n] == 7).all()          # nothing is written past the last row
    if added:
        assert ((dw[:n].double() - (want + 7)).abs() <= 2e-6 * scale + 1e-5).all()
    else:
        assert close(dw[:n], want, scale + 1e-3)


def test_without_a_workspace(g):
    import torch
    rows, n, k = 130, 136, 72
    assert K.linear_bwd_together(rows, n, k)
    dy, w, x = (torch.randn(*shape, device="cuda").bfloat16() for shape in ((rows, n), (n, k), (rows, k)))
    dx, dw = torch.empty_like(x), torch.empty_like(w)
    g.call(K.lib().karma_k_linear_bwd_bf16, g.ptr(dy), g.ptr(w), g.ptr(x), g.ptr(dx), g.ptr(dw), None, None, None, C.c_uint64(0), rows, n, k, 0,
           g.stream_ptr())
    assert close(dx, dy.double() @ w.double(), dy.double().abs() @ w.double().abs())
    assert close(dw, dy.double().T @ x.double(), dy.double().abs().T @ x.double().abs())
