"""Performance cases of the framework: fused CNN blocks and whole networks through `Session`.

Every case is one forward pass (`Session.run`) of a layer graph whose fusion blocks run as one
kernel each: the five benchmark configurations, the four fused structures of the paper's Table 1,
a batch-1 and a batch-64 network, an odd-sized block, and the split-bf16 operand mode.  A case is

    kind       which graph builder of xl_workloads makes it (see `_workload`)
    n          batch
    precision  0: fp32 matrix operations, 1: split-bf16 operands (xl_options.precision)
    tune       True: the program tunes its plan once with xl_tune, as bench.py and a serving program
               with a fixed shape do; False: the planner's own choice (a program that does not)
    ...        the sizes that builder takes

The path is inference only: there is no backward direction and no optimiser.
"""
import numpy as np
import torch

import xl_workloads as W

MAX_FLOPS = 12e9            # of a drawn case: below the batch-64 network (44.7e9)
MAX_ELEMENTS = 60_000_000   # of all tensors of a drawn case together


def listed():
    return [
        # The smallest call: two 3x3 layers on 16 channels of 16x16, one image; launch latency and host work.
        {"name": "straight_16x16_b1", "kind": "straight", "n": 1, "cin": 16, "h": 16, "w": 16, "c1": 16, "k1": 3,
         "c2": 16, "k2": 3, "precision": 0, "tune": False},
        # Pointwise convolution with folded batch normalisation and its max pooling, a small batch.
        {"name": "pool_56_b8", "kind": "pool", "n": 8, "cin": 64, "h": 56, "w": 56, "c1": 64, "k1": 1, "s1": 1,
         "pad_pool": 1, "precision": 0, "tune": True},
        # A SqueezeNet fire module (split mode) at a serving batch; 55x55 divides by no tile.
        {"name": "fire_55_b16", "kind": "fire", "n": 16, "cin": 96, "hw": 55, "s": 16, "e": 64, "precision": 0,
         "tune": True},
        # A residual basic block (merge mode), the arithmetic-heavy one.
        {"name": "residual_56_b32", "kind": "residual", "n": 32, "c": 64, "hw": 56, "precision": 0, "tune": True},
        # The same block on an odd number of odd-sized images and channels, on the planner's own choice.
        {"name": "residual_27_b5_c40", "kind": "residual", "n": 5, "c": 40, "hw": 27, "precision": 0, "tune": False},
        # Depthwise-separable pair (Table 1 a.2): bound by memory.
        {"name": "depthwise_80_b32", "kind": "depthwise", "n": 32, "c": 16, "h": 80, "w": 80, "c2": 16, "precision": 0,
         "tune": True},
        # Two 1x1 producers added into a 1x1 consumer (Table 1 c.1).
        {"name": "two_producers_56_b32", "kind": "two_producers", "n": 32, "c": 64, "h": 56, "w": 56, "cmid": 256,
         "cout": 64, "precision": 0, "tune": True},
        # 1x1 into 5x5 (Table 1 a.1).
        {"name": "conv5_28_b32", "kind": "straight", "n": 32, "cin": 192, "h": 28, "w": 28, "c1": 16, "k1": 1,
         "c2": 32, "k2": 5, "precision": 0, "tune": True},
        # The whole network for one image: interactive use, every launch is small.
        {"name": "net_224_b1", "kind": "net", "n": 1, "hw": 224, "classes": 1000, "precision": 0, "tune": True},
        # The whole network at the benchmark's batch: throughput, the largest case.
        {"name": "net_224_b64", "kind": "net", "n": 64, "hw": 224, "classes": 1000, "precision": 0, "tune": True},
        # The split-bf16 operand mode on the residual block and on the network at a serving batch.
        {"name": "residual_56_b32_bf16x3", "kind": "residual", "n": 32, "c": 64, "hw": 56, "precision": 1, "tune": True},
        {"name": "net_224_b8_bf16x3", "kind": "net", "n": 8, "hw": 224, "classes": 1000, "precision": 1, "tune": True},
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["straight", "straight5", "pool", "stem", "fire", "fire", "firepool", "residual", "residual", "head",
                       "depthwise", "two_producers", "net"])
    c = {"kind": kind, "n": _log_int(rng, 1, 64)}
    if kind == "straight":
        c.update(cin=_log_int(rng, 8, 96), h=rng.randint(8, 64), w=rng.randint(8, 64), c1=_log_int(rng, 8, 64),
                 k1=rng.choice([1, 3]), c2=_log_int(rng, 8, 96), k2=rng.choice([1, 3]))
    elif kind == "straight5":
        c.update(kind="straight", cin=_log_int(rng, 16, 192), h=rng.randint(12, 56), w=rng.randint(12, 56),
                 c1=_log_int(rng, 8, 32), k1=1, c2=_log_int(rng, 16, 64), k2=5)
    elif kind == "pool":
        c.update(cin=_log_int(rng, 8, 96), h=rng.randint(16, 112), w=rng.randint(16, 112), c1=_log_int(rng, 16, 64),
                 k1=rng.choice([1, 3]), s1=1, pad_pool=rng.choice([0, 1]))
    elif kind == "stem":
        c.update(kind="pool", cin=3, h=rng.randint(64, 256), w=rng.randint(64, 256), c1=_log_int(rng, 16, 96), k1=3, s1=2,
                 pad_pool=0)
    elif kind in ("fire", "firepool"):
        s = rng.choice([16, 24, 32, 48, 64])
        c.update(cin=_log_int(rng, 32, 512), hw=rng.randint(13, 56), s=s, e=rng.choice([2, 3, 4]) * s)
    elif kind == "residual":
        c.update(c=_log_int(rng, 16, 64), hw=rng.randint(9, 64))
    elif kind == "head":
        c.update(cin=_log_int(rng, 32, 512), h=rng.randint(5, 14), w=rng.randint(5, 14), classes=_log_int(rng, 10, 1000))
    elif kind == "depthwise":
        c.update(c=_log_int(rng, 8, 32), h=rng.randint(16, 112), w=rng.randint(16, 112), c2=_log_int(rng, 8, 64))
    elif kind == "two_producers":
        c.update(c=_log_int(rng, 16, 64), h=rng.randint(14, 56), w=rng.randint(14, 56), cmid=_log_int(rng, 32, 256),
                 cout=_log_int(rng, 16, 64))
    else:
        c.update(hw=rng.randint(96, 256), classes=_log_int(rng, 10, 1000))
    c["precision"] = 1 if rng.random() < 0.2 else 0
    c["tune"] = rng.random() < 0.7
    while c["n"] > 1 and (W.count_flops(_workload(c)) > MAX_FLOPS or _elements(_workload(c)) > MAX_ELEMENTS):
        c["n"] = max(1, c["n"] * 3 // 4)
    return c


def _workload(c):
    kind, n = c["kind"], c["n"]
    if kind == "straight":
        return W.straight_generic(n, c["cin"], c["h"], c["w"], c["c1"], c["k1"], c["k1"] // 2, 1, c["c2"], c["k2"],
                                  c["k2"] // 2, 1, dist="relu_normal")
    if kind == "pool":      # padding keeps the extent of a stride-1 layer; a strided (stem) layer has none
        pad = c["k1"] // 2 if c["s1"] == 1 else 0
        return W.conv_pool_generic(n, c["cin"], c["h"], c["w"], c["c1"], c["k1"], pad, c["s1"], 3, 2, c["pad_pool"],
                                   bn=c["s1"] == 1)
    if kind == "fire":
        return W.config(3, n=n, cin=c["cin"], hw=c["hw"], s=c["s"], e=c["e"])
    if kind == "firepool":
        return W.split_fire_pool(n=n, cin=c["cin"], hw=c["hw"], s=c["s"], e=c["e"])
    if kind == "residual":
        return W.config(4, n=n, c=c["c"], hw=c["hw"])
    if kind == "head":
        return W.conv_gap_generic(n, c["cin"], c["h"], c["w"], c["classes"], 1, 0, 1)
    if kind == "depthwise":
        return W.depthwise_pointwise(n, c["c"], c["h"], c["w"], c["c2"])
    if kind == "two_producers":
        return W.merge_two_producers(n, c=c["c"], h=c["h"], w=c["w"], cmid=c["cmid"], cout=c["cout"])
    if kind == "net":
        return W.config(5, n=n, hw=c["hw"], classes=c["classes"])
    raise ValueError(kind)


def _elements(wl):
    return sum(int(np.prod(s)) for s in wl.shapes)


def _tensors(wl, seed):
    """The input and the parameters, in the distributions of xl_workloads, drawn on the GPU."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)

    x = normal(*wl.shapes[wl.input_id])
    if wl.input_dist == "relu_normal":
        x = x.clamp_(min=0)
    params = {}
    for i, ly in enumerate(wl.layers):
        if ly.op != "conv":
            continue
        fan_in = ly.cin // ly.groups * ly.k * ly.k
        p = {"w": normal(ly.cout, ly.cin // ly.groups, ly.k, ly.k) * (2.0 / fan_in) ** 0.5, "scale": None, "shift": None}
        if ly.bn:
            p["scale"], p["shift"] = 1.0 + 0.1 * normal(ly.cout), 0.1 * normal(ly.cout)
        elif ly.bias:
            p["shift"] = 0.01 * normal(ly.cout)
        params[i] = p
    return x, params


def prepare(case, seed):
    from paper_2007_06000_amd.session import Session
    wl = _workload(case)
    x, params = _tensors(wl, seed)
    host = {i: {k: None if v is None else v.cpu().numpy() for k, v in p.items()} for i, p in params.items()}
    return {"session": Session(wl, x.cpu().numpy(), host, tune=case["tune"], precision=case["precision"])}


def run(state):
    return state["session"].run()


def work(case):
    """Block (or network) input, parameters and output once each; 2 * multiply-adds without halo recomputation."""
    wl = _workload(case)
    moved = int(np.prod(wl.shapes[wl.input_id])) + int(np.prod(wl.shapes[wl.output_id])) + W.count_params(wl)
    return {"bytes": 4.0 * moved, "flops": float(W.count_flops(wl))}


def tolerance(case):
    """About four times what was measured against `exact`: at most 3.3e-7 with fp32 operations, 6.4e-6 with split-bf16
    operands (relative 2-norm; the largest single difference is some ten times that)."""
    if case["precision"]:
        return {"rel": 3e-5, "max": 3e-4}
    return {"rel": 2e-6, "max": 2e-5}


def exact(case, seed):
    """The graph layer by layer in float64: a convolution is one matrix product per filter tap."""
    wl = _workload(case)
    x, params = _tensors(wl, seed)
    val = {wl.input_id: x.double()}
    for i, ly in enumerate(wl.layers):
        a = val[ly.inputs[0]]
        ho, wo = wl.shapes[ly.out][2:]
        if ly.op == "conv":
            p = {k: None if v is None else v.double() for k, v in params[i].items()}
            a = torch.nn.functional.pad(a, (ly.pad,) * 4)
            y = torch.zeros(wl.shapes[ly.out], dtype=torch.float64, device=a.device)
            for u in range(ly.k):
                for v in range(ly.k):
                    t = a[:, :, u:u + (ho - 1) * ly.stride + 1:ly.stride, v:v + (wo - 1) * ly.stride + 1:ly.stride]
                    if ly.groups != 1:
                        y += t * p["w"][:, 0, u, v].view(1, -1, 1, 1)
                    else:
                        f = p["w"][:, :, u, v].contiguous()
                        y += torch.matmul(f, t.reshape(t.shape[0], t.shape[1], -1).contiguous()).view_as(y)
            if p["scale"] is not None:
                y = y * p["scale"].view(1, -1, 1, 1)
            if p["shift"] is not None:
                y = y + p["shift"].view(1, -1, 1, 1)
        elif ly.op == "maxpool":
            y = torch.nn.functional.max_pool2d(a, ly.k, ly.stride, ly.pad)
        elif ly.op == "gap":
            y = a.mean(dim=(2, 3), keepdim=True)
        elif ly.op == "add":
            y = a + val[ly.inputs[1]]
        else:
            y = torch.cat([a, val[ly.inputs[1]]], dim=1)
        val[ly.out] = y.clamp(min=0) if ly.relu else y
    return val[wl.output_id]
