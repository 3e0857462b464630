"""The filter-gradient work that programs have this library do, as cases that can be timed.

A case is either one convolution layer through its own entry point, or one mini-batch of a network's layers
through a schedule run.  Sizes are those of the package's layer tables (CIFAR ResNet-20 and VGG-19) and, for
single layers, ordinary and odd ones around them.  Tensors are made on the GPU with the distributions of
``paper_1908_05460_amd.inputs``: X = max(z, 0), dY = 0.01 z.
"""
import math

import torch

from paper_1908_05460_amd import binding as B
from paper_1908_05460_amd import inputs, schedule

SCALE = 1.0 / 128                       # the paper's scale of the approximated gradient
STACKS = {"resnet20": inputs.resnet20_stack, "vgg19": inputs.vgg19_stack}
# one mini-batch's mask: (function of the schedule module, batch number)
MASKS = {"exact": (schedule.all_exact, 0), "approx": (schedule.alternate_batches, 1),
         "every_other": (schedule.every_other_layer, 0), "inner": (schedule.all_but_first_and_last, 0),
         "schedule1": (schedule.schedule1, 0)}


def _layer(name, method, dtype, n, c, k, h, w, r=3, s=3, stride=1, pad=1, topk=0):
    return {"name": name, "kind": "layer", "method": method, "dtype": dtype, "n": n, "c": c, "k": k, "h": h, "w": w,
            "r": r, "s": s, "stride": stride, "pad": pad, "topk": topk}


def _stack(name, net, mask, dtype, n):
    return {"name": name, "kind": "stack", "net": net, "mask": mask, "dtype": dtype, "n": n}


def listed():
    return [
        # one small layer at a time, as a program that calls the library per layer does: latency of a call
        _layer("layer_exact_small", "exact", "fp32", 16, 16, 16, 32, 32),
        _layer("layer_approx_small", "approx", "fp32", 16, 16, 16, 32, 32),
        # a layer that is no power of two anywhere
        _layer("layer_exact_odd", "exact", "fp32", 32, 48, 96, 27, 27),
        # a layer on image-sized planes
        _layer("layer_exact_image", "exact", "fp32", 4, 64, 64, 224, 224),
        # more than one kept position per map
        _layer("layer_top4", "topk", "fp32", 32, 64, 64, 56, 56, topk=4),
        # a training step of the small network: every gradient exact, every one approximated, and the last, shorter
        # mini-batch of an epoch (50 000 images in mini-batches of 128 leave 80) under a mixed schedule
        _stack("resnet20_exact", "resnet20", "exact", "fp32", 128),
        _stack("resnet20_approx", "resnet20", "approx", "fp32", 128),
        _stack("resnet20_every_other_n80", "resnet20", "every_other", "fp32", 80),
        # a training step of the large network
        _stack("vgg19_exact", "vgg19", "exact", "fp32", 128),
        _stack("vgg19_approx", "vgg19", "approx", "fp32", 128),
        # the same at a large mini-batch of bf16 tensors
        _stack("vgg19_bf16_exact", "vgg19", "exact", "bf16", 512),
        _stack("vgg19_bf16_approx", "vgg19", "approx", "bf16", 512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.4:
        dtype = rng.choice(["fp32", "fp32", "bf16"])
        return {"kind": "stack", "net": rng.choice(sorted(STACKS)), "mask": rng.choice(sorted(MASKS)), "dtype": dtype,
                "n": _log(rng, 16, 128 if dtype == "fp32" else 512)}
    while True:
        method = rng.choice(["exact", "exact", "approx", "approx", "topk"])
        dtype = rng.choice(["fp32", "fp32", "bf16"])
        if rng.random() < 0.5:          # a layer of a network whose channels double as its planes halve
            h = w = rng.choice([2, 4, 8, 16, 32, 56, 64])
            c = rng.choice([16, 32, 64, 128, 256, 512])
            k = c * rng.choice([1, 1, 2])
            r = s = 3
            stride, pad, n = 1 if k == c else rng.choice([1, 2]), 1, _log(rng, 8, 256)
        else:                           # any layer
            h, w = _log(rng, 5, 230), _log(rng, 5, 230)
            c, k = _log(rng, 3, 300), _log(rng, 8, 300)
            r = s = rng.choice([1, 3, 3, 3, 5])
            stride, pad, n = rng.choice([1, 1, 1, 2]), r // 2, _log(rng, 1, 100)
        case = _layer("", method, dtype, n, c, k, h, w, r, s, stride, pad)
        del case["name"]
        lay = _layer_of(case)
        if k > 512 or lay.flops(n) > 8e9 or n * max(c * h * w, k * lay.Ho * lay.Wo) > 2 ** 24 or lay.flops(n) < 1e7:
            continue
        if method == "topk":
            case["topk"] = min(rng.choice([2, 4, 8]), lay.Ho * lay.Wo)
        return case


def _layer_of(case):
    class Rect(inputs.Layer):           # the package's layers are square; a single call's need not be
        @property
        def Ho(self):
            return (case["h"] + 2 * self.pad - self.R) // self.stride + 1

        @property
        def Wo(self):
            return (case["w"] + 2 * self.pad - self.S) // self.stride + 1
    return Rect("layer", case["c"], case["k"], case["h"], case["w"], case["r"], case["s"], case["stride"], case["pad"])


def _layers(case):
    """[(layer, method)] of a case."""
    if case["kind"] == "layer":
        return [(_layer_of(case), case["method"])]
    layers = STACKS[case["net"]]()
    fn, batch = MASKS[case["mask"]]
    return [(l, schedule.METHOD_NAMES[int(m)]) for l, m in zip(layers, fn(len(layers), batch))]


def _tensors(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    out = []
    for l, _ in _layers(case):
        x = torch.randn((case["n"], l.C, l.H, l.W), generator=gen, device="cuda").clamp_(min=0).to(dt)
        dy = torch.randn((case["n"], l.K, l.Ho, l.Wo), generator=gen, device="cuda").mul_(inputs.DY_STD).to(dt)
        out.append((x, dy))
    return out


def prepare(case, seed):
    layers = _layers(case)
    tensors = _tensors(case, seed)
    descs = [B.desc_for(l, case["n"], case["dtype"]) for l, _ in layers]
    dws = [torch.empty((l.K, l.C, l.R, l.S), dtype=torch.float32, device="cuda") for l, _ in layers]
    state = {"case": case}
    if case["kind"] == "stack":
        fn, batch = MASKS[case["mask"]]
        methods = fn(len(layers), batch)
        run = B.Schedule(descs, [t[0] for t in tensors], [t[1] for t in tensors], dws)
        state.update(schedule=run, methods=methods, ws=B.alloc_workspace(run.workspace_bytes(methods)), dws=dws)
        return state
    d = descs[0]
    need = B.topk_workspace_bytes(d, case["topk"]) if case["method"] == "topk" else \
        B.workspace_bytes(d, B.EXACT if case["method"] == "exact" else B.APPROX)
    state.update(desc=d, x=tensors[0][0], dy=tensors[0][1], dw=dws[0], ws=B.alloc_workspace(need))
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "stack":
        state["schedule"].run(state["methods"], state["ws"], scale=SCALE)
        return state["dws"]
    args = state["desc"], state["x"], state["dy"]
    if case["method"] == "exact":
        return B.conv_wgrad_exact(*args, dW=state["dw"], ws=state["ws"])
    if case["method"] == "approx":
        return B.conv_wgrad_approx(*args, scale=SCALE, dW=state["dw"], ws=state["ws"])
    return B.conv_wgrad_approx_topk(*args, case["topk"], scale=SCALE, dW=state["dw"], ws=state["ws"])


def _valid(size, out, taps, stride, pad):
    return sum(1 for o in range(out) for t in range(taps) if 0 <= o * stride + t - pad < size)


def work(case):
    """Each input read once and each result written once; the multiply-adds whose tap lies inside X (of the kept
    positions only, for an approximated layer)."""
    size = 2 if case["dtype"] == "bf16" else 4
    n, nbytes, flops = case["n"], 0, 0
    for l, method in _layers(case):
        dw = l.K * l.C * l.R * l.S
        x = n * l.C * l.H * l.W
        nbytes += n * l.K * l.Ho * l.Wo * size + dw * 4
        if method == "exact":
            nbytes += x * size
            flops += 2 * n * l.K * l.C * _valid(l.H, l.Ho, l.R, l.stride, l.pad) * _valid(l.W, l.Wo, l.S, l.stride, l.pad)
        else:
            kept = max(1, case.get("topk", 0))
            nbytes += min(x, n * dw * kept) * size
            flops += 2 * n * dw * kept
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Four times the largest error against 64 bits that was seen over the listed cases and a few dozen drawn ones:
    9.7e-7 (largest entry 8.8e-6) where every product and sum is a 32-bit one, which for bf16 tensors the exact
    gradient's are too; 1.7e-3 (1.4e-2) where an approximated layer's map sums are rounded to bf16."""
    rounded = case["dtype"] == "bf16" and any(method != "exact" for _, method in _layers(case))
    return {"rel": 7e-3, "max": 6e-2} if rounded else {"rel": 4e-6, "max": 4e-5}


def _kept(dy, k, scale):
    """The approximated layer's dY: each map keeps its k largest magnitudes (the lowest index first among equals),
    each carrying an equal share of the map's sum."""
    n, c, h, w = dy.shape
    flat = dy.reshape(n * c, h * w)
    share = flat.sum(1) * (scale / k)
    if k == 1:
        mag = flat.abs()
        place = torch.arange(h * w, device=dy.device)
        at = torch.where(mag == mag.amax(1, keepdim=True), place, h * w).amin(1, keepdim=True)
    else:
        at = torch.sort(-flat.abs(), dim=1, stable=True).indices[:, :k]
    return torch.zeros_like(flat).scatter_(1, at, share[:, None].expand(-1, k)).reshape(dy.shape)


def _gradient(l, x, dy):
    """The definition, one filter tap at a time, in 64 bits."""
    n = x.shape[0]
    padded = torch.nn.functional.pad(x, (l.pad,) * 4)
    rows = dy.permute(1, 0, 2, 3).reshape(l.K, -1)
    dw = torch.empty((l.K, l.C, l.R, l.S), dtype=torch.float64, device=x.device)
    for r in range(l.R):
        for s in range(l.S):
            seen = padded[:, :, r:r + (l.Ho - 1) * l.stride + 1:l.stride, s:s + (l.Wo - 1) * l.stride + 1:l.stride]
            dw[:, :, r, s] = rows @ seen.permute(0, 2, 3, 1).reshape(n * l.Ho * l.Wo, l.C)
    return dw


def exact(case, seed):
    out = []
    for (l, method), (x, dy) in zip(_layers(case), _tensors(case, seed)):
        x, dy = x.double(), dy.double()
        if method != "exact":
            dy = _kept(dy, max(1, case.get("topk", 0)), SCALE)
        out.append(_gradient(l, x, dy))
    return out if case["kind"] == "stack" else out[0]
