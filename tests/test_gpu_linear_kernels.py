"""The fp32 layer of the MLP through karma_k_linear_relu_*: results that lie over inputs which the same call has no more use
for (the launches are ordered then) and sizes on both sides of the choice between the tiles, against float64 with the bounds
of fp32 sums of these lengths."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K
import synth_inputs as si


@pytest.fixture(scope="module")
def g():
    import gpu_util
    return gpu_util


def close(g, got, want, terms):
    """fp32 sums: 2^-24 per addition of a random walk, ten times that allowed"""
    return g.rel_l2(got, want) <= 10 * 2.0 ** -24 * np.sqrt(terms) or not np.any(want)


# what lies over what, and how much room the shared buffer needs
PLACES = [("dz", "z"), ("dz", "dy"), ("dx", "dy"), ("dx", "z"), ("dw", "dy"), ("dw", "z"), ("dw", "w"), ("db", "dy"), ("db", "z"),
          ("db", "w"), ("db", "x")]


@pytest.mark.parametrize("m,n,k", [(17, 64, 256), (260, 96, 40), (300, 520, 260)])
@pytest.mark.parametrize("out,over", PLACES)
def test_backward_results_over_inputs(g, m, n, k, out, over):
    import torch
    size = dict(x=(m, k), w=(n, k), z=(m, n), dy=(m, n), dz=(m, n), dx=(m, k), dw=(n, k), db=(n,))
    host = {name: si.normal(30 + i, size[name]).astype(np.float32) for i, name in enumerate(["x", "w", "z", "dy"])}
    dz = host["dy"].astype(np.float64) * (host["z"] > 0)
    want = dict(dz=dz, dx=dz @ host["w"].astype(np.float64), dw=dz.T @ host["x"].astype(np.float64), db=dz.sum(axis=0))
    room = {name: int(np.prod(s)) for name, s in size.items()}
    room[over] = max(room[over], room[out])
    buf = {name: torch.zeros(room[name], device="cuda") for name in size if name != out}
    buf[out] = buf[over]
    for name, a in host.items():
        buf[name][:a.size] = g.dev(a, torch.float32).reshape(-1)
    g.call(K.lib().karma_k_linear_relu_bwd_f32, *(g.ptr(buf[name]) for name in ("x", "w", "z", "dy", "dz", "dx", "dw", "db")), m, n, k,
           g.stream_ptr())
    for name, terms in (("dx", n), ("dw", m), ("db", m)):
        got = buf[name][:want[name].size].cpu().numpy().reshape(size[name])
        assert close(g, got, want[name], terms), name
    assert np.array_equal(buf["dz"][:m * n].cpu().numpy().reshape(m, n), dz.astype(np.float32))


# one size on either side of the choice between the tiles, forward and backward, with and without 16-byte rows (long
# reductions and many tiles take the large one), and edges of the large tile and of its 16 k
@pytest.mark.parametrize("m,n,k", [(1, 8, 8), (33, 65, 17), (1300, 1000, 30), (1300, 1000, 28), (400, 1441, 161), (420, 1440, 160), (700, 703, 1500),
                                   (96, 2309, 31), (1500, 1504, 1500)])
def test_both_tiles(g, m, n, k):
    import torch
    x, w, dy, b = (si.normal(40 + i, s).astype(np.float32) for i, s in enumerate([(m, k), (n, k), (m, n), (n,)]))
    xd, wd, dyd, bd = (g.dev(a, torch.float32) for a in (x, w, dy, b))
    z, y = torch.empty(m, n, device="cuda"), torch.empty(m, n, device="cuda")
    g.call(K.lib().karma_k_linear_relu_fwd_f32, g.ptr(xd), g.ptr(wd), g.ptr(bd), g.ptr(z), g.ptr(y), m, n, k, g.stream_ptr())
    assert close(g, z.cpu().numpy(), x.astype(np.float64) @ w.astype(np.float64).T + b, k)
    assert torch.equal(y, torch.where(z > 0, z, torch.zeros_like(z)))
    dz = dy.astype(np.float64) * (z.cpu().numpy() > 0)
    for with_dx in (True, False):
        out = dict(dz=torch.empty(m, n, device="cuda"), dx=torch.full((m, k), 7.0, device="cuda"), dw=torch.empty(n, k, device="cuda"),
                   db=torch.empty(n, device="cuda"))
        g.call(K.lib().karma_k_linear_relu_bwd_f32, g.ptr(xd), g.ptr(wd), g.ptr(z), g.ptr(dyd), g.ptr(out["dz"]),
               g.ptr(out["dx"]) if with_dx else None, g.ptr(out["dw"]), g.ptr(out["db"]), m, n, k, g.stream_ptr())
        assert np.array_equal(out["dz"].cpu().numpy(), dz.astype(np.float32))
        assert close(g, out["dw"].cpu().numpy(), dz.T @ x.astype(np.float64), m)
        assert close(g, out["db"].cpu().numpy(), dz.sum(axis=0), m)
        if with_dx:
            assert close(g, out["dx"].cpu().numpy(), dz @ w.astype(np.float64), n)
        else:
            assert (out["dx"] == 7).all()


def test_more_small_tiles_than_a_grid_holds(g):
    """2^20 x 4096 results are 2^24 tiles of 16 x 16, one more than a grid of 256-thread workgroups takes."""
    import torch
    m, n, k = 1 << 20, 4096, 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    x, w, b = (torch.randn(s, device="cuda", generator=gen) for s in ((m, k), (n, k), (n,)))
    z, y = torch.empty(m, n, device="cuda"), torch.empty(m, n, device="cuda")
    g.call(K.lib().karma_k_linear_relu_fwd_f32, g.ptr(x), g.ptr(w), g.ptr(b), g.ptr(z), g.ptr(y), m, n, k, g.stream_ptr())
    for rows in (slice(0, 40), slice(m // 2, m // 2 + 40), slice(m - 40, m)):
        want = x[rows].double() @ w.double().T + b.double()
        assert close(g, z[rows].cpu().numpy(), want.cpu().numpy(), k)
        assert torch.equal(y[rows], torch.where(z[rows] > 0, z[rows], torch.zeros_like(z[rows])))
