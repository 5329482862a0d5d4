"""Images on their way to the device: rounded to bf16 on the host (to nearest even, infinities and NaN kept), eight channels a
pixel there, zeros behind the image's own.  Sizes whose values are no whole 16-byte vectors, no whole workgroups of the kernel
that spreads the channels, and more than one part of the transfer.  The tensor is looked for in the slab, where it has to lie
at a multiple of 256 bytes, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import paper_2008_11421_amd as K
import synth_inputs as si


def stored(images, channels):
    u = np.ascontiguousarray(images, np.float32).reshape(-1, channels).view(np.uint32).astype(np.uint64)
    r = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    nan = (u & 0x7FFFFFFF) > 0x7F800000
    r[nan] = ((u[nan] >> 16) | 0x40).astype(np.uint16)
    out = np.zeros((len(r), 8), np.uint16)
    out[:, :channels] = r
    return out


CASES = [("unet", 1, 18), ("unet", 3, 38), ("unet", 2, 516), ("wrn", 1, 12), ("wrn", 7, 20), ("cnn", 5, 32)]


@pytest.mark.parametrize("kind,n,size", CASES)
def test_images_in_the_slab(kind, n, size):
    base = dict(n_layers=0, width=16, batch=n, seq=size, n_heads=0, ffn=0, vocab=8, stream_weights=0)
    if kind == "unet":
        desc = dict(base, kind=K.MODEL_UNET, n_layers=1, width=8)
    else:
        desc = dict(base, kind=K.MODEL_WRN if kind == "wrn" else K.MODEL_CNN, stage_blocks=(1, 1, 1, 0 if kind == "wrn" else 1))
    channels = 1 if kind == "unet" else 3
    cfg = dict(optimizer=K.OPT_SGD, lr=1e-3, beta1=0.0, beta2=0.0, eps=0.0, host_threads=3)
    layers, loss, fixed = K.karma_model_costs(desc, 490 * 10**12, 3 * 10**12)
    need = fixed + sum(l[3] + l[4] for l in layers) + 2 * max(max(l[5] for l in layers), loss[1]) + (32 << 20)
    ctx = K.Context(desc, cfg, need // 256 * 256)
    ctx.karma_set_plan(need // 256 * 256, [K.KEEP] * len(layers))
    images = si.normal(5, (n, size, size) if channels == 1 else (n, size, size, 3)).astype(np.float32)
    flat = images.reshape(-1)
    flat[:6] = [np.inf, -np.inf, np.nan, 1e-41, 3.4028235e38, -0.0]
    flat[-3:] = np.array([0x3F808000, 0x3F818000, 0x7F800001], np.uint32).view(np.float32)     # two ties and a signalling NaN
    labels = np.zeros((n, size, size) if channels == 1 else n, np.int32)
    ctx.karma_step(images, labels)
    want = stored(images, channels).reshape(-1)
    slab = ctx.arena[:fixed // 256 * 256].cpu().numpy().view(np.uint16)
    starts = np.arange(0, len(slab) - len(want) + 1, 128)
    for step in (0, 1, len(want) // 2, len(want) - 24):      # few offsets survive a look at some of the values
        starts = starts[slab[starts + step] == want[step]]
    assert any(np.array_equal(slab[s:s + len(want)], want) for s in starts)
    ctx.close()
