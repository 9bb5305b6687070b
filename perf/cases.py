"""Performance cases of the fused N-model training step.

A pass is what a training program does once per batch: `Hybrid.step` (or the
replay of a captured step) on the resident batch, for some cases preceded by
the hand-over of the next batch that already lies in device memory. Programs
that log every step read the per-model losses, which waits for the step; the
others only enqueue it.

The hybrids run on one stream of the program's own (`Hybrid.set_stream`), so
steps follow one another as the steps of one training do.

The updated parameters (and kept gradients, and optimizer state) stay on the
device, where the next step reads them. A pass returns them as `Trained`, which
copies them out of the context when they are looked up, as a program does when
its training ends; the work that computes them is enqueued by the pass itself.
"""
import math
import random

import numpy as np
import torch
import torch.nn.functional as F

from paper_2408_01331_amd import unifiednn as un
from paper_2408_01331_amd import workloads

R, POOL, FLAT, RB, RE = ("relu",), ("pool",), ("flatten",), ("res_begin",), ("res_end",)


def L(n):
    return ("linear", int(n))


def C(n, k, pad):
    return ("conv", int(n), int(k), int(pad))


# ---------------------------------------------------------------------------
# Cases. Keys: family (which builder below), arch (seed of the architecture
# draws), n (models), batch, prec ("f32", or "bf16" with fp32 master weights),
# opt ("sgd", "momentum", "adam"), losses (read every step), grads (kept and
# read, un_keep_grads), feed (a device-resident batch handed over before every
# step), graph (replay a captured step), rates (a learning rate per model), and
# the family's own sizes.
# ---------------------------------------------------------------------------
_BASE = dict(arch=0, opt="sgd", losses=False, grads=False, feed=False, graph=False, rates=False, lr=0.01)


def _case(**kw):
    return dict(_BASE, **kw)


def listed():
    return [
        # the smallest hybrid: two small fp32 MLPs whose program reads the
        # losses every step; launches and latency
        _case(name="mlp2_f32", family="workload", workload="mlp2", prec="f32", n=2, batch=64, losses=True),
        # eight MNIST-sized fp32 MLPs with their gradients kept (monitoring,
        # clipping): the usual small hybrid, its layers' gradients checked directly
        _case(name="mlp8_f32_grads", family="workload", workload="mlp8", prec="f32", n=8, batch=256, grads=True),
        # four LeNet-5: fp32 convolutions with channel counts that are no whole vectors
        _case(name="lenet4_f32", family="workload", workload="lenet4", prec="f32", n=4, batch=128, losses=True),
        # the largest hybrid: 64 ragged MLPs, 102 M parameters
        _case(name="mlp64_bf16", family="workload", workload="mlp64", prec="bf16", n=64, batch=512),
        # the most arithmetic: 16 CNNs
        _case(name="cifar16_bf16", family="workload", workload="cifar16", prec="bf16", n=16, batch=256),
        # small residual CNNs: unpooled convolutions, skips, a residual head
        _case(name="resnet8_bf16", family="workload", workload="resnet8", prec="bf16", n=8, batch=64),
        # transformer-style classifiers on 32 tokens
        _case(name="attn8_bf16", family="workload", workload="attn8", prec="bf16", n=8, batch=128),
        # ragged MLPs at odd sizes with Adam and a rate per model
        _case(name="mlp12_bf16_adam", family="mlp", prec="bf16", n=12, batch=200, feat=520, classes=37, depth_lo=2,
              depth_hi=4, width_lo=50, width_hi=900, opt="adam", rates=True, lr=1e-4, arch=3),
        # fp32 CNNs with whole-vector channels at a ragged batch, momentum, kept gradients
        _case(name="cnn4_f32_grads", family="cnn", prec="f32", n=4, batch=50, chan=3, side=32, kernel=3, blocks=2,
              width_lo=16, width_hi=40, step=4, classes=10, opt="momentum", grads=True, arch=1),
        # one attention layer and its MLP in fp32, odd sizes, kept gradients
        _case(name="attn5_f32_grads", family="attn", prec="f32", n=5, batch=37, tokens=24, tfeat=16, width_lo=24,
              width_hi=64, depth_lo=1, depth_hi=1, classes=7, grads=True, arch=2),
        # models on three datasets (images of two shapes and flat features) in one hybrid
        _case(name="groups7_bf16", family="groups", prec="bf16", n=7, batch=96, losses=True, arch=4),
        # a single wider MLP, its next batch handed over from device memory every step
        _case(name="mlp1_bf16_feed", family="mlp", prec="bf16", n=1, batch=256, feat=784, classes=10, depth_lo=4,
              depth_hi=4, width_lo=512, width_hi=1024, losses=True, feed=True, arch=5),
    ]


def _logint(rng, lo, hi):
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    """One more case of the same families and ranges, below the largest listed ones in work."""
    while True:
        fam = rng.choice(["mlp", "mlp", "cnn", "resnet", "attn", "groups"])
        c = _case(family=fam, arch=rng.randrange(1 << 30), prec=rng.choice(["f32", "bf16"]))
        c["opt"] = rng.choice(["sgd", "sgd", "sgd", "momentum", "adam"])
        if c["opt"] == "adam":
            c["lr"] = 1e-4
        c["losses"] = rng.random() < 0.5
        c["grads"] = rng.random() < 0.25
        c["rates"] = rng.random() < 0.2
        if fam == "mlp":
            c.update(n=_logint(rng, 1, 64), batch=_logint(rng, 16, 1200), feat=8 * _logint(rng, 8, 128),
                     classes=_logint(rng, 2, 130), depth_lo=2, depth_hi=rng.randint(2, 6), width_lo=_logint(rng, 16, 64),
                     width_hi=_logint(rng, 64, 2048))
            c["feed"] = rng.random() < 0.15
        elif fam == "cnn":
            c.update(n=_logint(rng, 1, 16), batch=_logint(rng, 16, 256), chan=rng.choice([1, 3]),
                     side=rng.choice([16, 20, 28, 32]), kernel=rng.choice([3, 5]), blocks=rng.randint(1, 3),
                     width_lo=_logint(rng, 6, 32), width_hi=_logint(rng, 32, 192), step=rng.choice([2, 4, 8, 16]),
                     classes=_logint(rng, 2, 100))
        elif fam == "resnet":
            c.update(n=_logint(rng, 1, 12), batch=_logint(rng, 16, 128), chan=3, side=rng.choice([16, 32]),
                     width_lo=16, width_hi=rng.choice([16, 32]), classes=10)
        elif fam == "attn":
            c.update(n=_logint(rng, 1, 10), batch=_logint(rng, 8, 160), tokens=rng.randint(4, 48),
                     tfeat=8 * rng.randint(1, 8), width_lo=8 * rng.randint(2, 8), width_hi=8 * rng.randint(8, 14),
                     depth_lo=1, depth_hi=rng.randint(1, 2), classes=_logint(rng, 2, 50))
        else:
            c.update(n=7, batch=_logint(rng, 24, 192))
        if fam != "groups" and c["opt"] == "sgd" and not c["feed"] and not c["rates"]:
            c["graph"] = rng.random() < 0.15
        flops = work(c)["flops"]
        odd = fam == "cnn" and c["step"] < 8 and c["prec"] == "bf16"  # channels that are no whole vectors
        cap = 2e10 if c["prec"] == "f32" or odd or fam == "attn" else 1.8e11
        if flops <= cap and _param_total(c) <= 5e7:
            return c


# ---------------------------------------------------------------------------
# Architectures
# ---------------------------------------------------------------------------
def _net(case):
    """(specs, input group of each model, [(batch, sample shape)] per group, init rule per model)."""
    rng = random.Random(case["arch"])
    fam, n, B = case["family"], case["n"], case["batch"]
    if fam == "workload":
        wl = workloads.get(case["workload"])
        return wl.specs, [0] * n, [(B, tuple(wl.in_shape))], [wl.init] * n
    if fam == "mlp":
        specs = []
        for _ in range(n):
            layers = []
            for _ in range(rng.randint(case["depth_lo"], case["depth_hi"]) - 1):
                layers += [L(_logint(rng, case["width_lo"], max(case["width_lo"], case["width_hi"]))), R]
            specs.append({"layers": layers + [L(case["classes"])], "num_classes": case["classes"]})
        return specs, [0] * n, [(B, (case["feat"],))], ["kaiming"] * n
    if fam == "cnn":
        specs, k, q = [], case["kernel"], case["step"]
        for _ in range(n):
            layers, side = [], case["side"]
            for j in range(case["blocks"]):
                w = _logint(rng, case["width_lo"], max(case["width_lo"], case["width_hi"]))
                w = max(q, w // q * q)
                side //= 2
                if j == case["blocks"] - 1:  # a Linear layer reads whole multiples of 8 features
                    while w * side * side % 8:
                        w += 1
                layers += [C(w, k, k // 2), R, POOL]
            specs.append({"layers": layers + [FLAT, L(case["classes"])], "num_classes": case["classes"]})
        return specs, [0] * n, [(B, (case["chan"], case["side"], case["side"]))], ["kaiming"] * n
    if fam == "resnet":
        specs = []
        for _ in range(n):
            c, h = rng.choice([case["width_lo"], case["width_hi"]]), rng.choice([64, 128])
            specs.append({"layers": _resnet(c, h, case["classes"]), "num_classes": case["classes"]})
        return specs, [0] * n, [(B, (case["chan"], case["side"], case["side"]))], ["torch"] * n
    if fam == "attn":
        specs = []
        for _ in range(n):
            w = 8 * rng.randint(case["width_lo"] // 8, max(case["width_lo"], case["width_hi"]) // 8)
            layers = [("unflatten", case["tokens"]), L(w), R]
            for _ in range(rng.randint(case["depth_lo"], case["depth_hi"])):
                layers += [RB, ("attention",), RE, R, RB, L(2 * w), R, L(w), RE, R]
            layers += [L(16), R, FLAT, L(case["classes"])]
            specs.append({"layers": layers, "num_classes": case["classes"]})
        return specs, [0] * n, [(B, (case["tokens"] * case["tfeat"],))], ["torch"] * n
    # groups: MNIST-shaped, CIFAR-shaped and flat inputs
    c1, c2, h = rng.choice([6, 8, 12]), rng.choice([16, 32]), rng.choice([37, 129, 300])
    specs = [
        {"layers": [C(c1, 5, 0), R, POOL, C(16, 5, 0), R, POOL, FLAT, L(120), R, L(10)], "num_classes": 10},
        {"layers": [FLAT, L(64), R, L(10)], "num_classes": 10},
        {"layers": [C(c2, 3, 1), R, POOL, C(2 * c2, 3, 1), R, POOL, FLAT, L(10)], "num_classes": 10},
        {"layers": [C(16, 3, 1), R, POOL, RB, C(16, 3, 1), RE, R, C(8, 3, 1), R, POOL, FLAT, L(10)], "num_classes": 10},
        {"layers": [L(h), R, L(129), R, L(13)], "num_classes": 13},
        {"layers": [L(200), R, L(13)], "num_classes": 13},
        {"layers": [L(13)], "num_classes": 13},
    ]
    inputs = [(B, (1, 28, 28)), (max(8, B // 2), (3, 32, 32)), (max(8, B // 3 + 5), (104,))]
    return specs, [0, 0, 1, 1, 2, 2, 2], inputs, ["torch"] * 7


def _resnet(c, h, classes):
    return [C(c, 3, 1), R, POOL, RB, C(c, 3, 1), R, C(c, 3, 1), RE, R, C(2 * c, 3, 1), R, POOL,
            RB, C(2 * c, 3, 1), R, C(2 * c, 3, 1), RE, R, C(2 * c, 3, 1), R, POOL, FLAT,
            L(h), R, RB, L(h), R, L(h), RE, R, L(classes)]


def _param_total(case):
    specs, group_of, inputs, _ = _net(case)
    return sum(int(np.prod(s)) for i, sp in enumerate(specs) for s, _ in workloads.param_shapes(sp, inputs[group_of[i]][1]))


def work(case):
    """Multiply-adds of forward, weight gradient and data gradient (none for a
    first layer), counted twice; bytes: the batch, the parameters read and
    written, and the optimizer state and kept gradients where there are any."""
    specs, group_of, inputs, _ = _net(case)
    flops, params = 0.0, 0
    for i, sp in enumerate(specs):
        B, shape = inputs[group_of[i]]
        first, tok = True, 1
        for l in sp["layers"]:
            m = 0.0
            if l[0] == "linear":
                seq = len(shape) == 2
                fin, tok = (shape[1], shape[0]) if seq else (int(np.prod(shape)), 1)
                m = float(B) * tok * fin * l[1]
                params += (fin + 1) * l[1]
                shape = (shape[0], l[1]) if seq else (l[1],)
            elif l[0] == "conv":
                c, h, w = shape
                oh, ow = h + 2 * l[3] - l[2] + 1, w + 2 * l[3] - l[2] + 1
                m = float(B) * oh * ow * c * l[2] * l[2] * l[1]
                params += (c * l[2] * l[2] + 1) * l[1]
                shape = (l[1], oh, ow)
            elif l[0] == "attention":
                T, d = shape
                m = float(B) * T * (4 * d * d + 2 * T * d)
                params += 4 * d * (d + 1)
            elif l[0] == "pool":
                shape = (shape[0], shape[1] // 2, shape[2] // 2)
            elif l[0] == "flatten":
                shape = (int(np.prod(shape)),)
            elif l[0] == "unflatten":
                shape = (l[1], shape[0] // l[1])
            if m:
                flops += 2 * m * (2 if first else 3)
                first = False
    state = {"sgd": 0, "momentum": 8, "adam": 16}[case["opt"]]
    nbytes = params * (8 + state + (4 if case["grads"] else 0))
    nbytes += sum(4 * B * (int(np.prod(s)) + 1) for B, s in inputs)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# Inputs, the pass
# ---------------------------------------------------------------------------
def _inputs(case, seed):
    """Flat parameters per model, (x, y) per input group, and the learning rates; host arrays, fp32."""
    specs, group_of, inputs, init = _net(case)
    rng = np.random.default_rng([seed, 77])
    theta = []
    for i, sp in enumerate(specs):
        parts = []
        for shape, fan_in in workloads.param_shapes(sp, inputs[group_of[i]][1]):
            kaiming = init[i] == "kaiming" and len(shape) > 1
            bound = np.float32(math.sqrt(6.0 / fan_in) if kaiming else 1.0 / math.sqrt(fan_in))
            u = rng.random(int(np.prod(shape)), dtype=np.float32)
            u *= 2 * bound
            u -= bound
            parts.append(u)
        theta.append(np.concatenate(parts))
    data = []
    for g, (B, shape) in enumerate(inputs):
        x = rng.standard_normal((B,) + tuple(shape), dtype=np.float32)
        classes = min(sp["num_classes"] for i, sp in enumerate(specs) if group_of[i] == g)
        data.append((x, rng.integers(0, classes, size=B).astype(np.int32)))
    n = len(specs)
    lrs = np.full(n, case["lr"], dtype=np.float32)
    if case["rates"]:
        lrs *= (1 + np.arange(n) % 4).astype(np.float32) / 2
    return theta, data, lrs


_stream = None


def _program_stream():
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream.cuda_stream


class Trained(dict):
    """What a pass leaves on the device, by name; copied out of the context when looked up."""

    def __init__(self, hybrid, names, losses):
        super().__init__({k: None for k in names})
        self.hybrid = hybrid
        if losses is not None:
            self["losses"] = losses

    def __getitem__(self, k):
        h = self.hybrid
        if k == "weights":
            return np.concatenate([h.get_params(i) for i in range(h.n)])
        if k == "grads":
            return np.concatenate([h.get_grads(i) for i in range(h.n)])
        if k == "state":
            return np.concatenate([h.get_opt_state(i)[0] for i in range(h.n)])
        return super().__getitem__(k)


def prepare(case, seed):
    specs, group_of, inputs, _ = _net(case)
    theta, data, lrs = _inputs(case, seed)
    if len(inputs) == 1:
        h = un.Hybrid(specs, inputs[0][0], inputs[0][1], case["prec"])
    else:
        h = un.Hybrid(specs, None, None, case["prec"], inputs=inputs, group_of=group_of)
    h.set_stream(_program_stream())
    for i, t in enumerate(theta):
        h.set_params(i, t)
        if case["opt"] == "momentum":
            h.set_optimizer(i, "momentum", momentum=0.9)
        elif case["opt"] == "adam":
            h.set_optimizer(i, "adam")
    for g, (x, y) in enumerate(data):
        h.load_batch(x, y, None if len(data) == 1 else g)
    if case["grads"]:
        h.keep_grads(True)
    state = {"hybrid": h, "lr": lrs if case["rates"] else case["lr"], "losses": case["losses"], "feed": None,
             "graph": case["graph"]}
    if case["feed"]:
        state["feed"] = tuple(torch.from_numpy(a).cuda() for a in data[0])
        torch.cuda.synchronize()
    if case["graph"]:
        h.capture(case["lr"])
    state["names"] = ["weights"] + (["grads"] if case["grads"] else []) + ([] if case["opt"] == "sgd" else ["state"])
    return state


def run(state):
    h = state["hybrid"]
    if state["feed"] is not None:
        x, y = state["feed"]
        un.un_load_batch_device(h.ctx, x.data_ptr(), y.data_ptr())
    if state["graph"]:
        losses = h.replay(losses=state["losses"])
    else:
        losses = h.step(state["lr"], losses=state["losses"])
    return Trained(h, state["names"], losses)


# ---------------------------------------------------------------------------
# Correctness
# ---------------------------------------------------------------------------
def tolerance(case):
    """About four times the errors measured against `exact` over the listed and
    some drawn cases. Updated weights hide most of a gradient's error, so a
    case that also returns gradients or optimizer state (which are gradients)
    has a wider one.
      f32:  weights 3e-8, losses 2e-7; gradients 4e-7, but two evaluation
            orders may decide a ReLU or a pool maximum within rounding of a tie
            differently, and one such unit and sample is about 2e-5 of a gradient
      bf16: weights 2.5e-4 (Adam 4e-4), losses 5.4e-4; gradients and state 0.03"""
    inner = case["grads"] or case["opt"] != "sgd"
    if case["prec"] == "f32":
        return {"rel": 1e-4 if inner else 1e-6}
    return {"rel": 0.12 if inner else 2e-3}


def _forward(spec, p, x):
    """Logits of one model, plain torch; p: its parameter tensors in state_dict order."""
    p = iter(p)
    h, skip = x, []
    for l in spec["layers"]:
        if l[0] == "linear":
            w, b = next(p), next(p)
            h = (h if h.dim() == 3 else h.flatten(1)) @ w.t() + b
        elif l[0] == "conv":
            w, b = next(p), next(p)
            n, _, hh, ww = h.shape
            k, pad = l[2], l[3]
            cols = F.unfold(h, k, padding=pad)  # [n, c k k, pixels]
            h = (w.flatten(1) @ cols + b[:, None]).view(n, l[1], hh + 2 * pad - k + 1, ww + 2 * pad - k + 1)
        elif l[0] == "attention":
            wi, bi, wo, bo = next(p), next(p), next(p), next(p)
            q, k, v = (h @ wi.t() + bi).chunk(3, dim=-1)
            a = torch.softmax(q @ k.transpose(1, 2).contiguous() / math.sqrt(h.shape[-1]), dim=-1)
            h = (a @ v.contiguous()) @ wo.t() + bo
        elif l[0] == "relu":
            h = torch.relu(h)
        elif l[0] == "pool":
            h = F.max_pool2d(h, 2)
        elif l[0] == "flatten":
            h = h.flatten(1)
        elif l[0] == "unflatten":
            h = h.view(h.shape[0], l[1], -1)
        elif l[0] == "res_begin":
            skip.append(h)
        elif l[0] == "res_end":
            h = h + skip.pop()
    return h


def exact(case, seed):
    specs, group_of, inputs, _ = _net(case)
    theta, data, lrs = _inputs(case, seed)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    losses, weights, grads, state = [], [], [], []
    for i, sp in enumerate(specs):
        x, y = (torch.from_numpy(a).to(dev) for a in data[group_of[i]])
        flat = torch.from_numpy(theta[i]).to(dev).double().requires_grad_()
        p, o = [], 0
        for shape, _ in workloads.param_shapes(sp, inputs[group_of[i]][1]):
            k = int(np.prod(shape))
            p.append(flat[o:o + k].view(shape))
            o += k
        loss = F.cross_entropy(_forward(sp, p, x.double()), y.long())
        g, = torch.autograd.grad(loss, flat)
        w, lr = flat.detach(), float(lrs[i])
        if case["opt"] == "adam":  # first step: the bias-corrected moments are g and g^2
            state += [0.1 * g, 0.001 * g * g]
            w = w - lr * g / (g.abs() + 1e-8)
        else:
            w = w - lr * g
            if case["opt"] == "momentum":
                state.append(g)
        losses.append(float(loss.detach()))
        weights.append(w.cpu())
        grads.append(g.cpu())
    out = {"weights": torch.cat(weights)}
    if case["grads"]:
        out["grads"] = torch.cat(grads)
    if case["opt"] != "sgd":
        out["state"] = torch.cat([s.cpu() for s in state])
    if case["losses"]:
        out["losses"] = np.array(losses)
    return out
