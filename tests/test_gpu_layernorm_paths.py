"""LayerNorm backward where its two forms meet: both sides of the choice, results that lie over inputs, as a caller may
place them once these are not needed any more, and more bands of rows than a grid's second dimension holds.  A bf16
result carries one rounding (2^-8 of the norm allowed); fp32 sums of n terms stay within n * 2^-24 of the terms."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def problem(rows, h, seed):
    """bf16 inputs on the device and, in float64, dx + add and the three column sums with the sums of their terms' sizes."""
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    make = lambda *s: torch.randn(s, device="cuda", generator=gen)
    x, dy, add = (make(rows, h) * 2 + 0.5).bfloat16(), make(rows, h).bfloat16(), make(rows, h).bfloat16()
    gamma = (1 + 0.2 * make(h)).bfloat16()
    mean = x.double().mean(1, keepdim=True)
    rstd = 1 / (x.double().var(1, unbiased=False, keepdim=True) + 1e-5).sqrt()
    stats = torch.cat([mean, rstd], 1).float()
    return x, dy, add, gamma, stats


def reference(x, dy, add, gamma, stats):
    xh = (x.double() - stats[:, :1].double()) * stats[:, 1:].double()
    t = dy.double() * gamma.double()
    dx = stats[:, 1:].double() * (t - t.mean(1, keepdim=True) - xh * (t * xh).mean(1, keepdim=True)) + add.double()
    sums = dict(dg=(dy.double() * xh), db=dy.double(), asum=add.double())
    return dx, {name: (v.sum(0), v.abs().sum(0)) for name, v in sums.items()}


def close_sums(got, want, rows):
    return bool(((got.double() - want[0]).abs() <= (rows + 4) * 2.0 ** -24 * want[1] + 1e-6).all())


def run(g, bufs, ws, rows, h):
    g.call(K.lib().karma_k_layernorm_bwd_addsum_bf16, *(g.ptr(bufs[n]) for n in ("dy", "x", "stats", "gamma", "add", "dx", "dg", "db", "asum")),
           g.ptr(ws), C.c_uint64(ws.numel() * 4), rows, h, g.stream_ptr())


# the pass that sums as it goes takes 12288 rows and more, from 8 Mi elements (10 Mi without add sums) and up to 3072 columns; else
# rows and columns are apart, in one launch, or in two where the gradient lies over an input and for 16 Mi elements of more columns:
# both sides of each line, each number of vectors per lane, last workgroups and last vectors that are not full
@pytest.mark.parametrize("rows,h", [(12288, 1032), (12291, 2056), (12300, 3072), (12287, 1032), (16385, 512), (16383, 512), (20483, 520),
                                    (12289, 3080), (40000, 264)])
@pytest.mark.parametrize("in_place", [False, True])
def test_one_pass_and_rows_apart_from_columns(g, rows, h, in_place):
    import torch
    x, dy, add, gamma, stats = problem(rows, h, rows + h)
    dx, sums = reference(x, dy, add, gamma, stats)
    ws = torch.empty((rows + 63) // 64 * 3 * h, device="cuda")
    lib, dim = K.lib(), (C.c_uint64(ws.numel() * 4), rows, h, g.stream_ptr())
    new = lambda: torch.full((h,), 7.0, device="cuda")
    plain = torch.empty_like(dy)
    dg, db = new(), new()
    g.call(lib.karma_k_layernorm_bwd_bf16, g.ptr(dy), g.ptr(x), g.ptr(stats), g.ptr(gamma), None, g.ptr(plain), g.ptr(dg), g.ptr(db),
           g.ptr(ws), *dim)
    assert ((plain.double() - (dx - add.double())).norm() / dx.norm()).item() <= 2.0 ** -8
    assert close_sums(dg, sums["dg"], rows) and close_sums(db, sums["db"], rows)
    out = dy if in_place else torch.empty_like(dy)
    bufs = dict(x=x, dy=dy, add=add, stats=stats, gamma=gamma, dx=out, dg=new(), db=new(), asum=new())
    run(g, bufs, ws, rows, h)
    err = (out.double() - dx).abs()
    assert (err.norm() / dx.norm()).item() <= 2.0 ** -8
    assert bool((err <= 2.0 ** -8 * dx.abs() + 1e-3 * dx.pow(2).mean(1, keepdim=True).sqrt()).all())
    for name in ("dg", "db", "asum"):
        assert close_sums(bufs[name], sums[name], rows), name


@pytest.mark.parametrize("rows,h", [(300, 264), (700, 264), (130, 4256), (16400, 776)])
@pytest.mark.parametrize("out", ["dg", "db", "asum"])
@pytest.mark.parametrize("over", ["dy", "x", "add", "stats", "gamma"])
def test_sums_over_inputs(g, rows, h, out, over):
    import torch
    x, dy, add, gamma, stats = problem(rows, h, rows + h)
    dx, sums = reference(x, dy, add, gamma, stats)
    bufs = dict(x=x, dy=dy, add=add, stats=stats, gamma=gamma, dx=torch.empty_like(x), dg=torch.empty(h, device="cuda"),
                db=torch.empty(h, device="cuda"), asum=torch.empty(h, device="cuda"))
    shared = torch.zeros(max(bufs[over].numel() * bufs[over].element_size(), 4 * h) // 4, device="cuda")
    bytes_of = lambda t: t.reshape(-1).view(torch.uint8)
    bytes_of(shared)[:bytes_of(bufs[over]).numel()] = bytes_of(bufs[over])
    bufs[over] = bufs[out] = shared
    ws = torch.empty((rows + 63) // 64 * 3 * h, device="cuda")
    run(g, bufs, ws, rows, h)
    assert ((bufs["dx"].double() - dx).norm() / dx.norm()).item() <= 2.0 ** -8
    for name in ("dg", "db", "asum"):
        assert close_sums(bufs[name][:h], sums[name], rows), name


def test_more_bands_than_a_second_grid_dimension_holds(g):
    """h above 3072 has rows and columns apart at any number of rows; 65536 bands of 64 rows and one row more."""
    import torch
    rows, h = 64 * 65536 + 1, 3080
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    x = torch.empty(rows, h, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    dy = torch.zeros_like(x)
    some = torch.tensor([0, 1, 63, 64, rows // 2, rows - 66, rows - 2, rows - 1], device="cuda")
    dy[some] = torch.randn(len(some), h, device="cuda", generator=gen).bfloat16()
    gamma = torch.randn(h, device="cuda", generator=gen).bfloat16()
    stats = torch.zeros(rows, 2, device="cuda")
    stats[:, 1] = 1
    mean = x[some].double().mean(1, keepdim=True)
    stats[some] = torch.cat([mean, 1 / (x[some].double().var(1, unbiased=False, keepdim=True) + 1e-5).sqrt()], 1).float()
    dx, sums = reference(x[some], dy[some], torch.zeros_like(dy[some]), gamma, stats[some])
    dg, db, ws = torch.empty(h, device="cuda"), torch.empty(h, device="cuda"), torch.empty((rows + 63) // 64 * 3 * h, device="cuda")
    g.call(K.lib().karma_k_layernorm_bwd_bf16, g.ptr(dy), g.ptr(x), g.ptr(stats), g.ptr(gamma), None, g.ptr(dy), g.ptr(dg), g.ptr(db),
           g.ptr(ws), C.c_uint64(ws.numel() * 4), rows, h, g.stream_ptr())
    assert ((dy[some].double() - dx).norm() / dx.norm()).item() <= 2.0 ** -8
    assert close_sums(dg, sums["dg"], len(some)) and close_sums(db, sums["db"], len(some))
    assert not dy[100].any() and not dy[rows - 100].any()
