"""The fp32 layer of the MLP through karma_k_linear_relu_*: results that lie over inputs which the same call has no more use
for (the launches are ordered then), against float64 with the bounds of fp32 sums of these lengths."""
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
