"""Performance cases: whole training steps and single layers through the library's public entry points.

A step case builds a context, loads seeded parameters, plans, and runs `karma_step` on a batch in host
memory, as a training loop does; it returns the loss and every parameter's gradient (where the optimiser
runs, the updated weights as well) as views of the device slab that the caller owns.  A layer case calls
the `karma_k_*` entry points of one layer, forward and backward, on device tensors.
"""
import ctypes as C
import math

import numpy as np
import torch

import paper_2008_11421_amd as K

MIB = 1 << 20


# ---------------------------------------------------------------------------------------- the listed cases
def listed():
    return [
        # The MLP of tests and benchmark (8 layers of 256, batch 32): the smallest step, all launches and host work.
        dict(name="mlp_step", kind="mlp", layers=8, width=256, batch=32),
        # A small transformer, as in a test or a first experiment: launches and small products.
        dict(name="gpt_small_step", kind="gpt", layers=3, hidden=256, heads=4, ffn=1024, vocab=2048, seq=256, batch=4, fit=100,
             optimizer=False),
        # The benchmark's transformer (hidden 1024, 16 heads of 64, batch 32 x 1024) cut to 4 of its 24 blocks, under a
        # budget that does not hold its activations (some halves recomputed or swapped), with the optimiser's update.
        dict(name="gpt_budget_step", kind="gpt", layers=4, hidden=1024, heads=16, ffn=4096, vocab=32000, seq=1024, batch=32, fit=60,
             optimizer=True),
        # One block of the 8.3B-parameter workload (24 heads of 128) at its batch, with a vocabulary cut in proportion.
        dict(name="gpt_heads128_step", kind="gpt", layers=1, hidden=3072, heads=24, ffn=12288, vocab=8192, seq=1024, batch=8,
             fit=100, optimizer=False),
        # One block of the 17B-parameter workload (28 heads of 152; no dimension is a whole number of tiles).
        dict(name="gpt_heads152_step", kind="gpt", layers=1, hidden=4256, heads=28, ffn=17024, vocab=8192, seq=1024, batch=4,
             fit=100, optimizer=False),
        # The bottleneck CNN at 224 x 224 with one block a stage (the projections and strides of every stage among them).
        dict(name="bottleneck_step", kind="cnn", width=64, blocks=1, image=224, batch=64, classes=1000),
        # The wide residual network at 32 x 32, one block a group.
        dict(name="wide_residual_step", kind="wrn", width=160, blocks=1, image=32, batch=256, classes=10),
        # The fully convolutional network: large images, few channels at the top, connections across.
        dict(name="unet_step", kind="unet", width=64, depth=3, image=256, batch=8, classes=2),
        # A classifier layer at a small batch (2048 -> 1000): the smallest products that a step has.
        dict(name="linear_classifier", kind="linear", rows=64, n_in=2048, n_out=1000, residual=False),
        # A projection of odd sizes with a residual: rows and widths that no tile divides.
        dict(name="linear_ragged", kind="linear", rows=3000, n_in=1416, n_out=2344, residual=True),
        # Self-attention on short sequences of a small batch.
        dict(name="attention_short", kind="attention", batch=4, seq=384, heads=12, d=64),
        # One strided convolution with its batch normalisation on an odd image.
        dict(name="conv_strided", kind="conv", batch=32, image=57, c_in=96, c_out=192, kernel=3, stride=2, relu=True),
    ]


def _log_int(rng, lo, hi, step=1):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def draw(rng):
    kind = rng.choice(["mlp", "gpt", "gpt", "gpt", "cnn", "wrn", "unet", "linear", "linear", "attention", "conv"])
    while True:
        case = _draw_one(rng, kind)
        w = work(case)
        if w["flops"] <= 8e12 and w["bytes"] <= 1.2e9:
            return case


def _draw_one(rng, kind):
    if kind == "mlp":
        return dict(kind=kind, layers=rng.randint(2, 12), width=_log_int(rng, 40, 512, 8), batch=_log_int(rng, 8, 128))
    if kind == "gpt":
        d = rng.choice([64, 64, 128, 152])
        heads = _log_int(rng, 2, {64: 20, 128: 26, 152: 28}[d])
        hidden = heads * d
        layers = rng.randint(1, 4)
        return dict(kind=kind, layers=layers, hidden=hidden, heads=heads,
                    ffn=rng.choice([4 * hidden, _log_int(rng, 2 * hidden, 4 * hidden, 8)]), vocab=_log_int(rng, 504, 16384, 8),
                    seq=128 * rng.randint(1, 8), batch=_log_int(rng, 1, 24), fit=rng.choice([100, 60]) if layers > 2 else 100, optimizer=False)
    if kind == "cnn":
        return dict(kind=kind, width=rng.choice([32, 64, 64]), blocks=1, image=32 * rng.randint(2, 8), batch=_log_int(rng, 4, 64),
                    classes=_log_int(rng, 104, 1000, 8))
    if kind == "wrn":
        return dict(kind=kind, width=16 * rng.randint(2, 10), blocks=1, image=4 * rng.randint(6, 16), batch=_log_int(rng, 16, 200),
                    classes=rng.choice([10, 100]))
    if kind == "unet":
        depth = rng.randint(2, 3)
        return dict(kind=kind, width=rng.choice([32, 64]), depth=depth, image=rng.randint(48, 320) >> depth << depth,
                    batch=_log_int(rng, 1, 8), classes=rng.choice([2, 6]))
    if kind == "linear":
        return dict(kind=kind, rows=_log_int(rng, 16, 8000, 4), n_in=_log_int(rng, 256, 4096, 8), n_out=_log_int(rng, 256, 4096, 8),
                    residual=rng.random() < 0.5)
    if kind == "attention":
        return dict(kind=kind, batch=_log_int(rng, 1, 8), seq=128 * rng.randint(1, 12), heads=rng.randint(1, 16),
                    d=rng.choice([64, 64, 128, 152]))
    k = rng.choice([1, 3, 3])
    return dict(kind="conv", batch=_log_int(rng, 4, 64), image=rng.randint(7, 112), c_in=_log_int(rng, 32, 320, 8),
                c_out=_log_int(rng, 32, 320, 8), kernel=k, stride=rng.choice([1, 1, 2]), relu=rng.random() < 0.7)


# ------------------------------------------------------------------------- models: tensors and what a step needs
# A model is a list of records, a record a list of (kind, shape): "matrix", "conv", "up" weights (gradients in
# bf16), "table" (the tied embedding, gradient in fp32), "gain", "shift", "bias" vectors (gradients in fp32).
def _conv(c_out, k, c_in):
    return ("conv", (c_out, k, k, c_in))


def _vec(c, kinds=("gain", "shift")):
    return [(k, (c,)) for k in kinds]


def _records(case):
    kind = case["kind"]
    if kind == "mlp":
        w = case["width"]
        return [[("matrix", (w, w)), ("bias", (w,))] for _ in range(case["layers"])] + [[]]
    if kind == "gpt":
        h, f = case["hidden"], case["ffn"]
        attn = _vec(h) + [("matrix", (3 * h, h)), ("bias", (3 * h,)), ("matrix", (h, h)), ("bias", (h,))]
        ffn = _vec(h) + [("matrix", (f, h)), ("bias", (f,)), ("matrix", (h, f)), ("bias", (h,))]
        return ([[("table", (case["vocab"], h)), ("matrix", (case["seq"], h))]] + [r for _ in range(case["layers"]) for r in (attn, ffn)]
                + [_vec(h)])
    if kind == "cnn":
        recs, c = [[_conv(case["width"], 7, 8)] + _vec(case["width"])], case["width"]
        for stage in range(4):
            m = case["width"] << stage
            for b in range(case["blocks"]):
                r = [_conv(m, 1, c)] + _vec(m) + [_conv(m, 3, m)] + _vec(m) + [_conv(4 * m, 1, m)] + _vec(4 * m)
                recs.append(r + ([_conv(4 * m, 1, c)] + _vec(4 * m) if b == 0 else []))
                c = 4 * m
        return recs + [[("matrix", (case["classes"], c)), ("bias", (case["classes"],))]]
    if kind == "wrn":
        recs, c = [[_conv(16, 3, 8)]], 16
        for group in range(3):
            m = case["width"] << group
            for b in range(case["blocks"]):
                r = _vec(c) + [_conv(m, 3, c)] + _vec(m) + [_conv(m, 3, m)]
                recs.append(r + ([_conv(m, 1, c)] if c != m else []))
                c = m
        return recs + [_vec(c) + [("matrix", (_stored(case), c)), ("bias", (_stored(case),))]]
    recs, c, w = [], 8, case["width"]
    for level in range(case["depth"] + 1):
        m = w << level
        recs.append([_conv(m, 3, c)] + _vec(m) + [_conv(m, 3, m)] + _vec(m))
        c = m
    for level in reversed(range(case["depth"])):
        m = w << level
        recs.append([("up", (2 * m, 2, 2, m)), _conv(m, 3, m), _conv(m, 3, m)] + _vec(m) + [_conv(m, 3, m)] + _vec(m))
    return recs + [[("matrix", (_stored(case), w)), ("bias", (_stored(case),))]]


def _stored(case):
    return (case["classes"] + 7) // 8 * 8       # class counts are stored in multiples of 8


def _conv_out(n, k, s, p):
    return (n + 2 * p - k) // s + 1


def _step_flops(case):
    """Multiply-adds of the forward products, twice that for the backward, two operations each."""
    kind, b = case["kind"], case["batch"]
    macs = 0
    if kind == "mlp":
        macs = case["layers"] * b * case["width"] ** 2
    elif kind == "gpt":
        h, t = case["hidden"], b * case["seq"]
        macs = t * (case["layers"] * (4 * h * h + 2 * h * case["ffn"] + case["seq"] * h) + h * case["vocab"])
    elif kind == "cnn":
        s = case["image"] // 2
        macs = s * s * case["width"] * 49 * 8
        s, c = s // 2, case["width"]
        for stage in range(4):
            m = case["width"] << stage
            for k in range(case["blocks"]):
                o = s // 2 if k == 0 and stage else s
                macs += s * s * c * m + o * o * (9 * m * m + 4 * m * m) + (o * o * c * 4 * m if k == 0 else 0)
                s, c = o, 4 * m
        macs = b * (macs + c * case["classes"])
    elif kind == "wrn":
        s, c = case["image"], 16
        macs = s * s * 16 * 9 * 8
        for group in range(3):
            m = case["width"] << group
            for k in range(case["blocks"]):
                o = _conv_out(s, 3, 2, 1) if k == 0 and group else s
                macs += o * o * (9 * c * m + 9 * m * m + (c * m if c != m else 0))
                s, c = o, m
        macs *= b
    else:
        for level in range(case["depth"] + 1):
            m, s = case["width"] << level, case["image"] >> level
            macs += s * s * 9 * m * ((m // 2 if level else 8) + m)
            if level < case["depth"]:
                macs += s * s * (2 * m * m + 27 * m * m)
        macs *= b
    return 6.0 * macs


def _input_bytes(case):
    if case["kind"] == "mlp":
        return 8 * case["batch"] * case["width"]
    if case["kind"] == "gpt":
        return 8 * case["batch"] * case["seq"]
    pixels = case["batch"] * case["image"] ** 2
    return pixels * 8 if case["kind"] == "unet" else pixels * 12 + 4 * case["batch"]


STEPS = ("mlp", "gpt", "cnn", "wrn", "unet")


def _out_size(case):
    return _conv_out(case["image"], case["kernel"], case["stride"], case["kernel"] // 2)


def work(case):
    kind = case["kind"]
    if kind in STEPS:      # weights read, gradients written, the batch read
        n = sum(int(np.prod(shape)) for rec in _records(case) for _, shape in rec)
        per = 8 if kind == "mlp" else 4
        if case.get("optimizer", True):      # fp32 master weights and their state read and written, new weights written
            per += {"mlp": 12, "gpt": 26}.get(kind, 18)
        return {"bytes": float(per * n + _input_bytes(case)), "flops": _step_flops(case)}
    if kind == "linear":
        m, n, k = case["rows"], case["n_out"], case["n_in"]
        return {"bytes": 2.0 * (2 * m * k + (3 if case["residual"] else 2) * m * n + 2 * n * k), "flops": 6.0 * m * n * k}
    if kind == "attention":
        rows, h = case["batch"] * case["seq"], case["heads"] * case["d"]
        return {"bytes": 2.0 * rows * h * (3 + 2 + 3), "flops": 2.0 * 3.5 * case["batch"] * h * case["seq"] ** 2}
    o = _out_size(case)
    x, y = case["batch"] * case["image"] ** 2 * case["c_in"], case["batch"] * o * o * case["c_out"]
    w = case["c_out"] * case["c_in"] * case["kernel"] ** 2
    return {"bytes": 2.0 * (2 * x + 2 * y + 2 * w), "flops": 6.0 * case["batch"] * o * o * w}


# --------------------------------------------------------------------------------------------------- preparing
class _Draw:
    """Seeded values, made on the GPU (a model's millions of weights) and handed over as the caller needs them."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, shape, std=1.0, mean=0.0):
        return torch.empty(shape, device="cuda", dtype=torch.float32).normal_(mean, std, generator=self.gen)

    def bf16(self, shape, std=1.0, mean=0.0):
        return self.normal(shape, std, mean).to(torch.bfloat16)

    def ints(self, shape, hi):
        return torch.randint(0, hi, shape, device="cuda", dtype=torch.int32, generator=self.gen)


def _weights(rnd, case, kind, shape, first, last):
    if kind == "gain":
        return rnd.normal(shape, 0.1, 1.0)
    if kind == "shift":
        return rnd.normal(shape, 0.1)
    if kind == "bias":
        v = rnd.normal(shape, 0.02)
        if last and case["kind"] in ("wrn", "unet"):
            v[case["classes"]:] = -30000.0            # the stored classes that do not exist
        return v
    if kind in ("conv", "up"):
        taps = shape[1] * shape[2]
        fan = shape[0] * taps if kind == "conv" else shape[3] * taps
        v = rnd.normal(shape, math.sqrt(2.0 / fan))
        if first:
            v[..., 1 if case["kind"] == "unet" else 3:] = 0.0   # image channels are stored as eight
        return v
    if case["kind"] == "mlp":
        return rnd.normal(shape, math.sqrt(1.0 / shape[0]))
    v = rnd.normal(shape, 0.02 if case["kind"] == "gpt" else 0.05)
    if last and case["kind"] in ("wrn", "unet"):
        v[case["classes"]:] = 0.0
    return v


def _desc(case):
    kind = case["kind"]
    d = dict(n_layers=0, width=case.get("width", 0), batch=case["batch"], seq=case.get("image", 0), n_heads=0, ffn=0, vocab=0,
             stream_weights=0)
    if kind == "mlp":
        d.update(kind=K.MODEL_MLP, n_layers=case["layers"])
    elif kind == "gpt":
        d.update(kind=K.MODEL_GPT, n_layers=case["layers"], width=case["hidden"], seq=case["seq"], n_heads=case["heads"],
                 ffn=case["ffn"], vocab=case["vocab"], split_blocks=1)
    elif kind == "cnn":
        d.update(kind=K.MODEL_CNN, vocab=case["classes"], stage_blocks=(case["blocks"],) * 4)
    elif kind == "wrn":
        d.update(kind=K.MODEL_WRN, vocab=_stored(case), stage_blocks=(case["blocks"],) * 3 + (0,))
    else:
        d.update(kind=K.MODEL_UNET, n_layers=case["depth"], vocab=_stored(case))
    return d


# Rates and link the plans are made with, so that a case has one plan on every machine and with every kernel:
# multiply-adds per second on the matrix cores, other operations per second; link bytes per second and latency.
RATES = (490 * 10**12, 3 * 10**12)
LINK = (57 * 10**9, 57 * 10**9, 8000)
# Update on the host as the backward pass goes (bottleneck network, MLP, most of the transformer) or, for the first
# records (all of them for the small networks), on the device.
SGD = dict(optimizer=K.OPT_SGD, lr=1e-3, beta1=0.0, beta2=0.0, eps=0.0)
MOMENTUM = dict(optimizer=K.OPT_SGD_MOMENTUM, lr=5e-3, beta1=0.9, beta2=0.0, eps=0.0)
ADAM = dict(optimizer=K.OPT_ADAM, lr=1e-4, beta1=0.9, beta2=0.999, eps=1e-8, device_update_first=3)
OPTIMISER = {"mlp": SGD, "gpt": ADAM, "cnn": MOMENTUM, "wrn": dict(MOMENTUM, device_update_first=99),
             "unet": dict(MOMENTUM, device_update_first=99)}
THREADS = 16


def _prepare_step(case, seed):
    rnd, records, desc = _Draw(seed), _records(case), _desc(case)
    layers, loss, fixed = K.karma_model_costs(desc, *RATES)
    optimise = case.get("optimizer", True)
    cfg = dict(OPTIMISER[case["kind"]] if optimise else SGD, host_threads=THREADS)
    on_device = min(cfg.get("device_update_first", 0), len(records) - 1)
    fixed += 12 * sum(int(np.prod(s)) + 64 for r in records[:on_device] for _, s in r)
    need = sum(l[3] + l[4] for l in layers) + 2 * max(max(l[5] for l in layers), loss[1])
    budget = (fixed + need * case.get("fit", 100) // 100 + 32 * MIB) // 256 * 256
    ctx = K.Context(desc, cfg, budget)
    off, weights, grads = 0, [], []
    up = lambda n: (n + 255) // 256 * 256
    for r, rec in enumerate(records):
        sizes = [int(np.prod(shape)) for _, shape in rec]
        for t, (kind, shape) in enumerate(rec):
            v = _weights(rnd, case, kind, shape, r == 0, r == len(records) - 1)
            ctx.karma_set_param(r, t, v.cpu().numpy())
        # the slab's fixed region: a record's weights, then its gradients, then optimiser state that lives there
        for (kind, shape), n in zip(rec, sizes):
            width = 4 if case["kind"] == "mlp" else 2
            weights.append(_view(ctx.arena, off, n, width).view(shape))
            off += up(n * width)
        for (kind, shape), n in zip(rec, sizes):
            width = 2 if case["kind"] != "mlp" and kind in ("matrix", "conv", "up") else 4
            grads.append(_view(ctx.arena, off, n, width).view(shape))
            off += up(n * width)
        if r < on_device:
            off += 3 * sum(up(4 * n) for n in sizes)
    ctx.karma_set_costs(layers, loss, LINK)
    ctx.karma_plan(budget)
    if case["kind"] == "mlp":
        batch = [rnd.normal((case["batch"], case["width"])) for _ in range(2)]
    elif case["kind"] == "gpt":
        batch = [rnd.ints((case["batch"], case["seq"]), case["vocab"]) for _ in range(2)]
    elif case["kind"] == "unet":
        n = case["image"]
        coarse = rnd.ints((case["batch"], -(-n // 16), -(-n // 16)), case["classes"])      # labels in patches, as masks have them
        label = coarse.repeat_interleave(16, 1).repeat_interleave(16, 2)[:, :n, :n].contiguous()
        batch = [rnd.normal((case["batch"], n, n)), label]
    else:
        batch = [rnd.normal((case["batch"], case["image"], case["image"], 3)), rnd.ints((case["batch"],), case["classes"])]
    return dict(kind="step", ctx=ctx, inputs=batch[0].cpu().numpy(), labels=batch[1].cpu().numpy(), optimise=optimise,
                out=_outputs(case, optimise, grads, weights))


def _outputs(case, optimise, grads, weights):
    """The transformer's and the MLP's gradients, and what the optimiser updated.  The convolutional networks give the
    updated weights alone: a batch normalisation before a ReLU leaves so many values near zero that two correct steps'
    gradients are far apart (0.1 to 0.4 of their norm), and the weights say as much as can be compared."""
    if case["kind"] in ("mlp", "gpt"):
        return [_joined(grads), _joined(weights, matrices=True)] if optimise else [_joined(grads)]
    return [_joined(weights)]


def _view(slab, off, n, width):
    return slab[off:off + n * width].view(torch.float32 if width == 4 else torch.bfloat16)


def _joined(views, matrices=False):
    """Vectors (or, with matrices, tensors) that lie side by side in the slab and hold one type, as one tensor."""
    out = []
    for v in views:
        last = out[-1] if out else None
        if (last is not None and v.dtype == last.dtype and (matrices or v.dim() == last.dim() == 1)
                and last.data_ptr() + last.element_size() * last.numel() == v.data_ptr()):
            out[-1] = torch.as_strided(last, (last.numel() + v.numel(),), (1,))
        else:
            out.append(v)
    return out


def _prepare_linear(case, seed):
    rnd, m, n, k = _Draw(seed), case["rows"], case["n_out"], case["n_in"]
    new = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    return dict(kind="linear", m=m, n=n, k=k, x=rnd.bf16((m, k)), w=rnd.bf16((n, k), 0.02), b=rnd.bf16((n,), 0.02),
                res=rnd.bf16((m, n)) if case["residual"] else None, dy=rnd.bf16((m, n), 0.1), y=new(m, n), dx=new(m, k), dw=new(n, k),
                ws=torch.empty(64 * MIB, dtype=torch.uint8, device="cuda"))


def _prepare_attention(case, seed):
    rnd, b, s, heads, d = _Draw(seed), case["batch"], case["seq"], case["heads"], case["d"]
    h = heads * d
    f32 = lambda n: torch.empty(n, dtype=torch.float32, device="cuda")
    return dict(kind="attention", dims=(b, s, heads, d), qkv=rnd.bf16((b, s, 3 * h)), dctx=rnd.bf16((b, s, h), 0.1),
                ctx=torch.empty((b, s, h), dtype=torch.bfloat16, device="cuda"), lse=f32(b * heads * s), delta=f32(b * heads * s),
                dqkv=torch.empty((b, s, 3 * h), dtype=torch.bfloat16, device="cuda"), dbias=f32(3 * h), ws=f32(b * s // 32 * 3 * h))


def _prepare_conv(case, seed):
    rnd, b, s, ci, co, k = _Draw(seed), case["batch"], case["image"], case["c_in"], case["c_out"], case["kernel"]
    o = _out_size(case)
    rows = b * o * o
    new = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    f32 = lambda n: torch.empty(n, dtype=torch.float32, device="cuda")
    return dict(kind="conv", shape=K.binding.ConvShape(b, s, s, ci, co, k, k, case["stride"], k // 2), rows=rows, c=co,
                relu=int(case["relu"]), x=rnd.bf16((b, s, s, ci)), w=rnd.bf16((co, k, k, ci), math.sqrt(2.0 / (co * k * k))),
                gain=rnd.bf16((co,), 0.1, 1.0), shift=rnd.bf16((co,), 0.1), da=rnd.bf16((b, o, o, co)),
                y=new(b, o, o, co), a=new(b, o, o, co), dy=new(b, o, o, co), dx=new(b, s, s, ci), dw=new(co, k, k, ci),
                stats=f32(2 * co), dgain=f32(co), dshift=f32(co), wt=new(k * k * ci * co), ws=f32(16 * k * k * ci * co),
                bn_ws=torch.empty(_bn_ws_bytes(rows, co), dtype=torch.uint8, device="cuda"))


def _bn_ws_bytes(rows, c):
    fn = K.lib().karma_k_batchnorm_ws_bytes
    fn.restype = C.c_uint64
    return int(fn(C.c_uint32(rows), C.c_uint32(c)))


def prepare(case, seed):
    kind = case["kind"]
    if kind in STEPS:
        return _prepare_step(case, seed)
    return {"linear": _prepare_linear, "attention": _prepare_attention, "conv": _prepare_conv}[kind](case, seed)


# ----------------------------------------------------------------------------------------------------- one pass
def _p(t):
    return C.c_void_p(t.data_ptr()) if t is not None else None


def _call(fn, *args):
    st = fn(*args)
    if st:
        raise RuntimeError("%s: status %d" % (fn.__name__, st))


def _run_step(s):
    loss = s["ctx"].karma_step(s["inputs"], s["labels"], K.STEP_APPLY_OPTIMIZER if s["optimise"] else 0)
    if s["optimise"]:
        s["ctx"].karma_finish_updates()
    return [loss, s["out"]]


def _run_linear(s):
    """y = x w^T + b (+ residual), dx = dy w, dw = dy^T x."""
    f, m, n, k = K.lib().karma_k_gemm_bf16, s["m"], s["n"], s["k"]
    ws, size, q = _p(s["ws"]), C.c_uint64(s["ws"].numel()), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    _call(f, _p(s["x"]), _p(s["w"]), _p(s["y"]), _p(s["b"]), _p(s["res"]), m, n, k, 0, ws, size, q)
    _call(f, _p(s["dy"]), _p(s["w"]), _p(s["dx"]), None, None, m, k, n, K.GEMM_B_STRIDED, ws, size, q)
    _call(f, _p(s["dy"]), _p(s["x"]), _p(s["dw"]), None, None, n, k, m, K.GEMM_A_STRIDED | K.GEMM_B_STRIDED, ws, size, q)
    return [s["y"], s["dx"], s["dw"]]


def _run_attention(s):
    lib, (b, n, heads, d) = K.lib(), s["dims"]
    q = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    _call(lib.karma_k_attention_fwd_bf16, _p(s["qkv"]), _p(s["ctx"]), _p(s["lse"]), b, n, heads, d, q)
    _call(lib.karma_k_attention_bwd_colsum_bf16, _p(s["qkv"]), _p(s["ctx"]), _p(s["dctx"]), _p(s["lse"]), _p(s["delta"]), _p(s["dqkv"]),
          _p(s["dbias"]), _p(s["ws"]), C.c_uint64(s["ws"].numel() * 4), b, n, heads, d, q)
    return [s["ctx"], s["lse"], s["dqkv"], s["dbias"]]


def _run_conv(s):
    lib, shape = K.lib(), C.byref(s["shape"])
    q = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    _call(lib.karma_k_conv2d_fwd_bf16, _p(s["x"]), _p(s["w"]), _p(s["y"]), shape, q)
    _call(lib.karma_k_batchnorm_fwd_bf16, _p(s["y"]), _p(s["gain"]), _p(s["shift"]), None, _p(s["a"]), _p(s["stats"]), _p(s["bn_ws"]),
          s["rows"], s["c"], s["relu"], q)
    _call(lib.karma_k_batchnorm_bwd_bf16, _p(s["da"]), _p(s["y"]), _p(s["stats"]), _p(s["gain"]), _p(s["shift"]), s["relu"], _p(s["dy"]),
          _p(s["dgain"]), _p(s["dshift"]), _p(s["bn_ws"]), s["rows"], s["c"], q)
    _call(lib.karma_k_conv2d_wgrad_bf16, _p(s["dy"]), _p(s["x"]), _p(s["dw"]), _p(s["ws"]), C.c_uint64(s["ws"].numel() * 4), shape, q)
    _call(lib.karma_k_conv2d_dgrad_bf16, _p(s["dy"]), _p(s["w"]), _p(s["wt"]), None, _p(s["dx"]), shape, q)
    return [s["y"], s["a"], s["dx"], s["dw"], s["dgain"], s["dshift"]]


def run(state):
    return {"step": _run_step, "linear": _run_linear, "attention": _run_attention, "conv": _run_conv}[state["kind"]](state)


def tolerance(case):
    """About four times what the same pass shows with its sums in another order (or, for the steps, with weights that
    differ by 2^-20 of themselves, which moves a few roundings in every layer)."""
    kind = case["kind"]
    if kind == "mlp":           # fp32 sums: 2.7e-6, 3e-5
        return {"rel": 1e-5, "max": 2e-4}
    if kind == "gpt":           # bf16 tensors through every layer: 8e-3, 0.15
        return {"rel": 3e-2, "max": 0.5}
    if kind in STEPS:           # the update's share of the weights, whose gradients are far apart: 5e-3, 0.1
        return {"rel": 2e-2, "max": 0.5}
    if kind == "linear":        # against fp32 products: 7e-5, one rounding of an element
        return {"rel": 3e-4, "max": 0.03}
    if kind == "attention":     # against fp32: 2.7e-3 (probabilities and their gradients are rounded to bf16), 0.1
        return {"rel": 1e-2, "max": 0.4}
    return {"rel": 2e-3, "max": 0.2}      # convolution, normalisation and back, against fp32: 3e-4, 0.05
