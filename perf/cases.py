"""The work that this framework does for its users, as cases to be timed.

Most cases are training steps through `lpp.Context` (a snapshot of the shared
replica, a forward pass, a backward pass cut off at a block, the block's
momentum update), on networks of `models.py` or on a few of their units; the
rest are the stand-alone kernels (replica averaging, block update, snapshot).
A step case makes `updates` updates with each of its workers and then fetches
what a training program looks at: logits, the last gradient, the parameters.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2203_06638_amd import lpp
from paper_2203_06638_amd import models as PM


# ---------------------------------------------------------------------------
# the cases

# The learning rate where a schedule has annealed to almost nothing.  At a larger one the rounding differences of one
# update, and the order in which updaters that share a replica meet, grow from update to update until two right
# answers no longer look alike (measured: 6% on ResNet-20's gradients after eight updates of four updaters at 1e-4).
LR = 1e-5


def _step(name, net, batch, **kw):
    """A step case; the fields every network kind understands.

    dtype    fp32, or bf16 activations and conv weights with fp32 masters
    mode     async: calls return at once (how training runs); sequential:
             every call waits, batch-norm sums in a fixed order (how runs are
             checked against each other)
    workers  one: a single updater; all: every updater of every replica, each
             on its own stream, steps on its own block
    full     the whole model's gradient (partition 0) instead of the block's
    """
    c = {"name": name, "kind": "step", "net": net, "batch": batch, "hw": 32, "classes": 10, "width": 16, "units": 3,
         "stages": 3, "dtype": "fp32", "mode": "async", "replicas": 1, "workers": "one", "full": True, "updates": 8,
         "lr": LR, "weight_decay": 0.0}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a tiny CNN's last block on 8 images, waited for (launches and latency only)
        _step("tiny_b8_sequential", "tiny", 8, mode="sequential", full=False, updates=1, width=8),
        # the benchmark's workload: ResNet-20, four updaters of one replica on four streams, each on its block
        _step("resnet20_b128_4_updaters", "resnet20", 128, workers="all", full=False),
        # a deterministic run of whole-model steps at a small batch, 100 classes
        _step("resnet20_b32_sequential", "resnet20", 32, classes=100, mode="sequential", updates=4),
        # small images of another size than the benchmark's, a batch that is no power of two, weight decay
        _step("resnet20_28px_b100", "resnet20", 100, hw=28, updates=4, weight_decay=5e-4),
        # the first half of an ImageNet ResNet at full precision (7x7 stem, 3x3/2 pool, units at 56 and 28 pixels)
        _step("imagenet_units_b16", "imagenet", 16, hw=224, width=64, units=2, stages=2, classes=100, updates=2),
        # one unit of each of these stages in mixed precision at a training batch
        _step("imagenet_units_b64_bf16", "imagenet", 64, hw=224, width=64, units=1, stages=2, classes=100, updates=4,
              dtype="bf16"),
        # bottleneck units at 28 pixels, the batch that the framework's ResNet-50 trains with
        _step("bottleneck_units_b32_bf16", "bottleneck", 32, hw=112, width=128, units=2, stages=1, classes=100,
              updates=4, dtype="bf16"),
        # biased convs without batch norm, concatenations, a pooled 1x1 conv as the classifier
        _step("squeezenet_b128", "squeezenet", 128, updates=4),
        # two replicas of four updaters each, averaged after four updates of every updater
        _step("wrn16_8_b128_2_replicas_bf16", "wrn16_8", 128, classes=100, workers="all", full=False, replicas=2,
              updates=4, dtype="bf16"),
        # an averaging round over four replicas of ResNet-18's size
        {"name": "average_4_replicas", "kind": "average", "n": 11689512, "replicas": 4},
        # the block update of a whole ResNet-50, momentum and weight decay
        {"name": "update_resnet50", "kind": "update", "n": 25557032, "momentum": 0.9, "weight_decay": 1e-4},
        # the snapshot of WRN-16-8 with its cast to bf16
        {"name": "snapshot_wrn16_8_bf16", "kind": "snapshot", "net": "wrn16_8", "classes": 100, "hw": 32, "width": 16,
         "units": 2, "stages": 3, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["cifar", "cifar", "imagenet", "imagenet", "bottleneck", "squeezenet", "resnet20", "average",
                       "update", "snapshot"])
    if kind == "average":
        return {"kind": kind, "n": _log(rng, 300000, 26000000), "replicas": rng.randint(2, 6)}
    if kind == "update":
        return {"kind": kind, "n": _log(rng, 300000, 26000000), "momentum": rng.choice([0.0, 0.9]),
                "weight_decay": rng.choice([0.0, 1e-4])}
    if kind == "snapshot":
        return {"kind": kind, "net": rng.choice(["imagenet", "bottleneck"]), "classes": rng.randint(10, 200), "hw": 64,
                "width": 8 * rng.randint(1, 32), "units": rng.randint(1, 3), "stages": 3,
                "dtype": rng.choice(["fp32", "bf16"])}
    kw = {"mode": "sequential" if rng.random() < 0.25 else "async", "classes": rng.randint(10, 120),
          "updates": rng.randint(2, 4), "weight_decay": rng.choice([0.0, 5e-4])}
    # (bf16 nets of a few layers at batches of 16 and more: in deeper ones, and at smaller batches, two right gradients
    # are further apart than a comparison can allow)
    if kind == "resnet20":      # several updaters, any batch and image size
        kw.update(workers="all", full=False, mode="async", hw=rng.choice([32, rng.randint(24, 48)]))
        c = _step("", kind, _log(rng, 16, 160), **kw)
    elif kind == "cifar":
        kw.update(hw=rng.randint(16, 48), width=4 * rng.randint(4, 12), units=rng.randint(1, 3))
        c = _step("", kind, _log(rng, 8, 160), **kw)
    elif kind == "imagenet" and rng.random() < 0.5:
        kw.update(hw=rng.randint(64, 224), width=8 * rng.randint(4, 10), units=rng.randint(1, 2), stages=rng.randint(1, 3))
        c = _step("", kind, _log(rng, 4, 16), **kw)
    elif kind == "imagenet":
        kw.update(hw=rng.randint(96, 224), width=8 * rng.randint(4, 24), units=rng.randint(1, 2), stages=1, dtype="bf16")
        c = _step("", kind, _log(rng, 16, 64), **kw)
    elif kind == "bottleneck":
        kw.update(hw=rng.randint(64, 160), width=8 * rng.randint(4, 32), units=1, stages=1, dtype="bf16")
        c = _step("", kind, _log(rng, 16, 64), **kw)
    else:
        kw.update(hw=rng.randint(24, 48), classes=4 * rng.randint(3, 30))    # (its logits come in fours)
        c = _step("", kind, _log(rng, 8, 128), **kw)
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs

def _model(c):
    net, n, hw, w, u = c["net"], c["classes"], c["hw"], c["width"], c["units"]
    if net == "tiny":
        return PM.tiny_cnn(n, hw)
    if net == "resnet20":       # the benchmark's four blocks, at any image size
        blocks = [1, 1, 1, 2, 2, 3, 3, 3, 4, 4, 4] if c["workers"] == "all" else None
        return PM.resnet_cifar(20, (16, 32, 64), n, hw, blocks)
    if net == "cifar":
        return PM.resnet_cifar(6 * u + 2, (w, 2 * w, 4 * w), n, hw)
    if net == "wrn16_8":
        return PM.wrn16_8(n)
    widths = tuple(w * 2 ** i for i in range(c["stages"]))
    if net == "imagenet":
        return PM.resnet_imagenet((u,) * c["stages"], widths, n, hw)
    if net == "bottleneck":
        return PM.resnet_bottleneck((u,) * c["stages"], widths, n, hw)
    return PM.squeezenet(n, hw)


def _generator(seed, k=0):
    return torch.Generator("cuda").manual_seed(int(seed) * 1000003 + k)


def _params(model, seed):
    """He-normal conv weights, uniform linear weights, batch-norm scales about
    1 and shifts and biases about 0 (their spread is that of a net in
    training)."""
    g = _generator(seed, 1)
    parts = []
    for kind, n, fan_in in model.specs:
        if kind == "conv_w":
            parts.append(torch.randn(n, generator=g, device="cuda") * math.sqrt(2.0 / fan_in))
        elif kind == "linear_w":
            parts.append((torch.rand(n, generator=g, device="cuda") * 2 - 1) / math.sqrt(fan_in))
        else:
            parts.append(torch.randn(n, generator=g, device="cuda") * 0.05 + (1.0 if kind == "bn_gamma" else 0.0))
    return torch.cat(parts)


def _batches(c, model, seed, count):
    out = []
    for k in range(count):
        g = _generator(seed, 10 + k)
        img = torch.randn((c["batch"],) + model.in_shape, generator=g, device="cuda")
        if c["dtype"] == "bf16":
            img = img.bfloat16().float()
        lab = torch.randint(model.n_classes, (c["batch"],), generator=g, device="cuda", dtype=torch.int32)
        out.append((img, lab))
    return out


def _snapshot_convs(model, bf16):
    """The conv tensors of a parameter vector and where their two kernel
    layouts go, as lpp.SnapshotPlan takes them; the vector's length and the
    layout buffer's."""
    vec = 8 if bf16 else 4
    convs, pos, wf = [], 0, 0
    for op, in0, _, cin, cout, k, _, _, bias, _ in model.layers:
        if op == lpp.CONV:
            cin_p = -(-cin // vec) * vec if in0 < 0 else cin
            nf, nd = -(-cout * k * k * cin_p // 64) * 64, -(-cin * k * k * cout // 64) * 64
            convs.append((pos, cout, cin, cin_p, k, k, wf, wf + nf))
            wf += nf + nd
            pos += cout * cin * k * k + (cout if bias else 0)
        elif op == lpp.BN:
            pos += 2 * cout
        elif op == lpp.LINEAR:
            pos += cout * cin + cout
    return convs, pos, wf


MOMENTUM = 0.9
BATCHES = 2     # minibatches in device memory that the updates take in turn


def _workers(c, model):
    """(worker, partition) in the order in which a round issues them"""
    if c["workers"] == "all":
        return [(w, w % model.P + 1) for w in range(c["replicas"] * model.P)]
    if c["net"] == "tiny":
        return [(1, 2)]
    return [(0, 0 if c["full"] else 1)]


def prepare(case, seed):
    c = case
    if c["kind"] == "average":
        g = _generator(seed)
        x = torch.randn(c["n"], generator=g, device="cuda")     # replicas have drifted a little apart
        reps = [x + 0.01 * torch.randn(c["n"], generator=g, device="cuda") for _ in range(c["replicas"])]
        return {"case": c, "reps": reps}
    if c["kind"] == "update":
        g = _generator(seed)
        x, m, grad = (s * torch.randn(c["n"], generator=g, device="cuda") for s in (0.05, 1e-3, 1e-3))
        return {"case": c, "x": x, "m": m if c["momentum"] else None, "g": grad}
    model = _model(c)
    x = _params(model, seed)
    bf16 = c["dtype"] == "bf16"
    if c["kind"] == "snapshot":
        convs, d, wf = _snapshot_convs(model, bf16)
        return {"case": c, "x": x, "v": torch.zeros(d, device="cuda"),
                "w": torch.zeros(wf, device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32),
                "plan": lpp.SnapshotPlan(convs, d, lpp.BF16 if bf16 else lpp.FP32, wf)}
    ctx = lpp.Context(model, c["replicas"], c["batch"], mode=lpp.SEQUENTIAL if c["mode"] == "sequential" else lpp.ASYNC,
                      dtype=lpp.BF16 if bf16 else lpp.FP32, momentum=MOMENTUM, weight_decay=c["weight_decay"])
    ctx.set_params(x.cpu().numpy())
    batches = _batches(c, model, seed, BATCHES)
    torch.cuda.synchronize()    # the inputs are there before the context's own streams read them
    return {"case": c, "ctx": ctx, "batches": batches, "workers": _workers(c, model)}


# ---------------------------------------------------------------------------
# one pass

def run(state):
    c = state["case"]
    if c["kind"] == "average":
        lpp.kernel_average(state["reps"])
        return state["reps"]
    if c["kind"] == "update":
        lpp.kernel_sgd_update(state["x"], state["m"], state["g"], 0.01, c["momentum"], c["weight_decay"])
        return [state["x"], state["m"]] if c["momentum"] else [state["x"]]
    if c["kind"] == "snapshot":
        state["plan"].run(state["x"], state["v"], state["w"])
        return [state["v"], state["w"]]
    ctx, workers, batches = state["ctx"], state["workers"], state["batches"]
    for u in range(c["updates"]):
        img, lab = batches[u % len(batches)]
        for w, part in workers:
            ctx.step(w, img, lab, part, c["lr"])
    if c["replicas"] > 1:
        ctx.sync()              # the round begins when every updater has made its updates
        ctx.average()
    # (of several updaters the last one's gradient, that of the last block: the others' lie behind more ReLUs, and in
    # bf16 the order in which the updaters met shows there; of several replicas one: they agree after the average)
    return {"logits": [ctx.get_logits(w) for w, _ in workers], "params": [ctx.get_params(0)],
            "grad": [ctx.get_grad(workers[-1][0])]}


def work(case):
    c = case
    if c["kind"] == "average":
        return {"bytes": 8.0 * c["n"] * c["replicas"], "flops": 3.0 * c["n"] * c["replicas"]}
    if c["kind"] == "update":
        return {"bytes": (20.0 if c["momentum"] else 12.0) * c["n"], "flops": 6.0 * c["n"]}
    model = _model(c)
    if c["kind"] == "snapshot":
        eb = 2 if c["dtype"] == "bf16" else 4
        conv = sum(n for kind, n, _ in model.specs if kind == "conv_w")
        return {"bytes": (4.0 + 2 * eb) * conv + 8.0 * (model.d - conv), "flops": 0.0}
    info = lpp.describe(model, c["batch"], dtype=lpp.BF16 if c["dtype"] == "bf16" else lpp.FP32)
    img = c["batch"] * (4.0 * math.prod(model.in_shape) + 4.0)
    flops = nbytes = 0.0
    for _, part in _workers(c, model):
        block = info.block_hi[part] - info.block_lo[part]
        flops += info.fwd_flops + info.bwd_flops[part]
        # the batch and the replica read; the block's momentum read and written, its parameters and gradient written
        nbytes += img + 4.0 * model.d + 16.0 * block + 4.0 * c["batch"] * model.n_classes
    nbytes, flops = nbytes * c["updates"], flops * c["updates"]
    if c["replicas"] > 1:
        nbytes += 8.0 * model.d * c["replicas"]
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Steps: the gradient decides.  It jumps wherever an input of a ReLU lies
    so close to zero that two roundings disagree about its sign: the same
    inputs with their images in another order give gradients up to 4e-3 apart
    in fp32 (logits 2e-6) and 2.2e-2 in bf16 (logits 7e-4); two runs of the
    bf16 updaters that share a replica give 2.6e-2 (logits 3e-3)."""
    c = case
    if c["kind"] in ("average", "update"):
        return {"rel": 1e-6, "max": 1e-5}
    if c["kind"] == "snapshot":
        return "exact"
    if c["dtype"] == "bf16":
        return {"rel": 3e-2, "max": 0.99}
    if c["net"] == "tiny":      # its last block has no ReLU behind it
        return {"rel": 2e-6, "max": 2e-5}
    return {"rel": 1.6e-2, "max": 0.99}


# ---------------------------------------------------------------------------
# the same in 64 bits

def _exact_step(model, x, img, lab, part, eps=1e-5):
    """logits and gradient of the mean cross-entropy with respect to block
    `part` (0: all) at parameters x, from the layer list in plain torch."""
    import torch.nn.functional as F
    x = x.detach().requires_grad_(True)
    outs, pos, lo, hi = [], 0, None, 0

    def take(n):
        nonlocal pos
        pos += n
        return x[pos - n:pos]

    for op, in0, in1, cin, cout, k, stride, pad, bias, block in model.layers:
        a = img if in0 < 0 else outs[in0]
        start = pos
        if op == lpp.CONV:
            w = take(cout * cin * k * k).view(cout, cin, k, k)
            y = F.conv2d(a, w, take(cout) if bias else None, stride, pad)
        elif op == lpp.BN:
            mean, var = a.mean((0, 2, 3), keepdim=True), a.var((0, 2, 3), unbiased=False, keepdim=True)
            y = (a - mean) * torch.rsqrt(var + eps) * take(cout).view(1, -1, 1, 1) + take(cout).view(1, -1, 1, 1)
        elif op == lpp.RELU:
            y = torch.relu(a)
        elif op == lpp.ADD:
            y = a + outs[in1]
        elif op == lpp.CONCAT:
            y = torch.cat([a, outs[in1]], 1)
        elif op == lpp.MAXPOOL:
            y = F.max_pool2d(a, k, stride, pad)
        elif op == lpp.GAP:
            y = a.mean((2, 3), keepdim=True)
        else:
            y = (a.flatten(1) @ take(cout * cin).view(cout, cin).t() + take(cout))[:, :, None, None]
        outs.append(y)
        if pos > start and part in (0, block):
            lo, hi = start if lo is None else lo, pos
    logits = outs[-1].flatten(1)
    grad, = torch.autograd.grad(F.cross_entropy(logits, lab.long()), x)
    block_only = torch.zeros_like(grad)
    block_only[lo:hi] = grad[lo:hi]
    return logits.detach(), block_only, lo, hi


def exact(case, seed):
    c = case
    if c["kind"] == "average":
        s = prepare(c, seed)
        mean = sum(r.double() for r in s["reps"]) / c["replicas"]
        return [mean] * c["replicas"]
    if c["kind"] == "update":
        s = prepare(c, seed)
        x, g = s["x"].double(), s["g"].double()
        m = g + float(np.float32(c["weight_decay"])) * x
        if c["momentum"]:
            m += float(np.float32(c["momentum"])) * s["m"].double()
        x -= float(np.float32(0.01)) * m
        return [x, m] if c["momentum"] else [x]
    model = _model(c)
    x = _params(model, seed).double()
    if c["kind"] == "snapshot":
        convs, d, wf = _snapshot_convs(model, c["dtype"] == "bf16")
        v, w = x.clone(), torch.zeros(wf, device="cuda", dtype=torch.float64)
        for src, cout, cin, cin_p, kh, kw, f, dg in convs:
            n = cout * cin * kh * kw
            t = x[src:src + n].view(cout, cin, kh, kw)
            v[src:src + n] = 0
            wide = torch.zeros(cout, kh, kw, cin_p, device="cuda", dtype=torch.float64)
            wide[..., :cin] = t.permute(0, 2, 3, 1)
            w[f:f + wide.numel()] = wide.flatten()
            w[dg:dg + n] = t.permute(1, 2, 3, 0).flatten()
        return [v, w]
    if c["workers"] == "all":
        return None     # updaters that share a replica without locks: every interleaving is a right answer
    (_, part), = _workers(c, model)
    m = torch.zeros_like(x)
    batches = [(i.double(), t) for i, t in _batches(c, model, seed, BATCHES)]
    for u in range(c["updates"]):
        img, lab = batches[u % BATCHES]
        logits, g, lo, hi = _exact_step(model, x, img, lab, part)
        m[lo:hi] = MOMENTUM * m[lo:hi] + g[lo:hi] + c["weight_decay"] * x[lo:hi]
        x[lo:hi] -= c["lr"] * m[lo:hi]
    # at fp32 a gradient's distance from 64 bits is that of a few ReLU inputs that 32 bits cannot tell from zero
    # (1e-6 or 1e-3, by which way they fall), and says nothing about how exactly the sums were formed
    jumps = c["dtype"] != "bf16" and c["net"] != "tiny"
    return {"logits": [logits], "params": [x], "grad": [None if jumps else g]}
