"""Kernels whose waves divide the reductions (variants 350 to 362 and 550 to 562) against the oracle: filter sizes, strides and
paddings of either layer, channels that fill neither K steps nor row tiles, tiles over the image's edge, poolings with padding."""
import numpy as np
import pytest

import xl_workloads as W
from oracle import xlo


def named(wl, name):
    wl.name = name
    return wl


def residual(n, c, h, w, k1, k2):
    b = W._Builder(f"res_{c}_{k1}_{k2}", n, c, h, w)
    t = b.conv(0, 40, k1, pad=k1 // 2, bn=True, relu=True, name="conv1")
    t = b.conv(t, c, k2, pad=k2 // 2, bn=True, relu=False, name="conv2")
    b.add(t, 0, relu=True, name="add")
    b.group("merge", 0)
    return b.done(len(b.shapes) - 1, "relu_normal", 31)


CASES = [
    named(W.config(3, n=1, hw=13, cin=512, s=64, e=256), "fire_512"), named(W.config(3, n=2, hw=9, cin=37, s=16, e=48), "fire_37"),
    named(W.config(3, n=1, hw=20, cin=130, s=48, e=96), "fire_130"), named(W.config(3, n=1, hw=5, cin=8, s=24, e=33), "fire_8"),
    named(W.split_fire_pool(n=2, cin=64, hw=15, s=16, e=64), "firepool_64"), named(W.split_fire_pool(n=1, cin=200, hw=13, s=64, e=100, pp=1), "firepool_200"),
    named(W.split_fire_pool(n=1, cin=90, hw=19, s=48, e=64), "firepool_90"),
    residual(2, 40, 17, 13, 3, 3), residual(1, 64, 27, 27, 3, 3), residual(2, 24, 9, 11, 1, 3), residual(1, 70, 12, 10, 1, 1),
    W.straight_generic(1, 16, 16, 16, 16, 3, 1, 1, 16, 3, 1, 1), W.straight_generic(2, 24, 17, 19, 70, 3, 1, 2, 48, 3, 1, 1),
    W.straight_generic(1, 24, 19, 21, 40, 3, 2, 1, 48, 3, 0, 2), W.straight_generic(1, 40, 19, 21, 16, 1, 0, 1, 32, 5, 3, 2),
    W.straight_generic(1, 130, 14, 15, 17, 1, 0, 1, 40, 5, 2, 1),
    W.straight_generic(1, 9, 15, 11, 9, 3, 1, 1, 22, 5, 2, 1), W.straight_generic(3, 50, 11, 9, 31, 1, 0, 2, 64, 3, 1, 1),
]


def candidates(p, base):
    out = {}
    for c in range(p.num_candidates(True, 0)):
        v = p.candidate_info(True, 0, c)["variant"]
        if base <= v < base + 13:
            out.setdefault(v - base, []).append(c)
    return out


def test_every_kernel_is_planned():
    from paper_2007_06000_amd import binding as B
    for precision, base in ((0, 550), (1, 350)):
        seen = set()
        for wl in CASES:
            got = candidates(B.Plan(wl, precision=precision), base)
            assert got, wl.name
            seen |= set(got)
        assert seen == set(range(13)), (precision, set(range(13)) - seen)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("wl", CASES, ids=lambda a: getattr(a, "name", ""))
def test_against_the_oracle(wl, precision):
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    s = Session(wl, x, params, precision=precision)
    for v, cs in candidates(s.plan, 350 if precision else 550).items():
        for c in cs:
            print(f"[case] {wl.name} kernel {v} candidate {s.plan.candidate_info(True, 0, c)}", flush=True)
            s.plan.select_candidate(True, 0, c)
            y = s.output(True)
            # three parts: sums of up to 1600 terms of random sign in up to nine pieces and two roundings per layer, 2^-20 is 16
            # of them; two parts: 3 * 2^-16 of the absolute sums at most, here within four times that of the result's norm
            assert np.linalg.norm(y - ref) <= (2.0 ** -12 if precision else 2.0 ** -20) * np.linalg.norm(ref), (v, c)


@pytest.mark.gpu
@pytest.mark.parametrize("special", [np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("wl", CASES, ids=lambda a: getattr(a, "name", ""))
def test_values_without_bf16_parts(wl, special):
    """One such value, in the input and in a filter of either layer: what the fp32 kernels make of it, and nothing else changes."""
    from paper_2007_06000_amd.session import Session
    convs = [i for i, ly in enumerate(wl.layers) if ly.op == "conv"]
    for where in [None] + convs:
        x, params = W.make_tensors(wl)
        if where is None:
            x[0, 1, x.shape[2] // 2, x.shape[3] // 2] = special
        else:
            w = params[where]["w"]
            w[3, min(5, w.shape[1] - 1), w.shape[2] // 2, w.shape[3] // 2] = special
        s = Session(wl, x, params)
        fp32 = [c for c in range(s.plan.num_candidates(True, 0)) if s.plan.candidate_info(True, 0, c)["variant"] < 200][0]
        s.plan.select_candidate(True, 0, fp32)
        ref = s.output(True)
        fin = np.isfinite(ref) & (np.abs(ref) < 1e20)
        for v, cs in candidates(s.plan, 550).items():
            print(f"[case] {wl.name} {special} in {where} kernel {v} candidate {s.plan.candidate_info(True, 0, cs[0])}", flush=True)
            s.plan.select_candidate(True, 0, cs[0])
            y = s.output(True)
            assert (np.isnan(y) == np.isnan(ref)).all() and (np.isfinite(y) == np.isfinite(ref)).all(), (where, v)
            assert (np.abs(y[fin] - ref[fin]) <= 1e-4 + 1e-4 * np.abs(ref[fin])).all(), (where, v)


@pytest.mark.gpu
@pytest.mark.parametrize("special", [3.4e38, 2.0 ** -134])
@pytest.mark.parametrize("wl", [wl for wl in CASES if wl.layers[0].k == 1], ids=lambda a: getattr(a, "name", ""))
def test_values_without_bf16_parts_in_pointwise_first_layers_on_two_parts(wl, special):
    """Layer 1 takes three parts there too: such a value in the input and in its filter, with finite sums, which is what two parts hold."""
    from test_gpu_chain import against_fp32_operations_on_two_parts
    value = np.float32(special) * np.float32(1 + 2.0 ** -10 if special < 1 else 1)
    for where in ("x", "w"):
        x, params = W.make_tensors(wl)
        if where == "x":
            x[0, 1, x.shape[2] // 2, x.shape[3] // 2] = value
            params[0]["w"] *= np.float32(0.25)          # sums below 2^127
        else:
            x *= np.float32(0.1)
            params[0]["w"][3, 5, 0, 0] = value
        if params[0]["scale"] is not None:
            params[0]["scale"][:] = 1.0
        assert against_fp32_operations_on_two_parts(wl, x, params, 350, 9, f"{special} in {where}")


def siblings(cin, hw, s, e1, e3):
    b = W._Builder(f"siblings_{cin}_{s}_{e1}_{e3}", 1, cin, hw, hw)
    sq = b.conv(0, s, 1, bias=True, relu=True, name="squeeze")
    a = b.conv(sq, e1, 1, bias=True, relu=True, name="expand1x1")
    c = b.conv(sq, e3, 3, pad=1, bias=True, relu=True, name="expand3x3")
    t = b.concat(a, c, name="concat")
    b.group("split", 0)
    return b.done(t, "relu_normal", 37)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("wl", [siblings(64, 9, 32, 160, 256), siblings(64, 9, 32, 256, 160), siblings(40, 11, 48, 33, 300)],
                         ids=lambda a: getattr(a, "name", ""))
def test_slices_without_rows_of_one_sibling(wl, precision):
    """Four slices of 5 and 8, or 2 and 10, row tiles: a workgroup that has rows of one sibling only."""
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    s = Session(wl, x, params, precision=precision, force_cout_split=4)
    found = candidates(s.plan, 350 if precision else 550)
    assert found
    for v, cs in found.items():
        for c in cs:
            print(f"[case] {wl.name} kernel {v} candidate {s.plan.candidate_info(True, 0, c)}", flush=True)
            s.plan.select_candidate(True, 0, c)
            y = s.output(True)
            # (bounds as in test_against_the_oracle)
            assert np.linalg.norm(y - ref) <= (2.0 ** -12 if precision else 2.0 ** -20) * np.linalg.norm(ref), (v, c)


def in_64_bits(wl, x, params):
    """The graph's convolutions and additions without a rounding."""
    import torch
    val = {wl.input_id: torch.from_numpy(x).double()}
    for i, ly in enumerate(wl.layers):
        a = val[ly.inputs[0]]
        if ly.op == "conv":
            p = {k: None if v is None else torch.from_numpy(v).double() for k, v in params[i].items()}
            y = torch.nn.functional.conv2d(a, p["w"], None, ly.stride, ly.pad)
            for key, apply in (("scale", torch.mul), ("shift", torch.add)):
                if p.get(key) is not None:
                    y = apply(y, p[key].view(1, -1, 1, 1))
        else:
            assert ly.op == "add"
            y = a + val[ly.inputs[1]]
        val[ly.out] = y.clamp(min=0) if ly.relu else y
    return val[wl.output_id].numpy()


@pytest.mark.gpu
@pytest.mark.parametrize("wl", [W.config(4, n=3, c=19, hw=29), W.config(4, n=4, c=17, hw=30), W.config(4, n=1, c=18, hw=47), W.config(4, n=2, c=28, hw=45)],
                         ids=["19", "17", "18", "28"])
def test_error_is_no_larger_than_that_of_the_general_kernels_on_parts(wl):
    """Short reductions in eight parts, where the roundings of adding them up weigh most."""
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = in_64_bits(wl, x, params)
    s = Session(wl, x, params)
    err = {}
    for c in range(s.plan.num_candidates(True, 0)):
        v = s.plan.candidate_info(True, 0, c)["variant"]
        if v < 400 or v in err:
            continue
        s.plan.select_candidate(True, 0, c)
        err[v] = np.linalg.norm(s.output(True) - ref) / np.linalg.norm(ref)
    mine, general = [e for v, e in err.items() if v >= 550], [e for v, e in err.items() if v < 520]
    assert mine and general
    # (norms over 39000 or more outputs: 0.5 % between orders of the same sums, 2 % is four times that)
    assert max(mine) <= 1.02 * min(general), err
