"""Kernels on operands in three bf16 parts (variants from 400 in a plan of fp32 precision) against the kernels on fp32
matrix operations: no less exact, and the same results for values that do not come apart into bf16 parts."""
import numpy as np
import pytest

import xl_workloads as W
from oracle import xlo

pytestmark = pytest.mark.gpu

FIRST, END = 400, 600       # variant ids of the kernels under test

WORKLOADS = [
    W.single_conv(2, 40, 9, 31, 70, 3, 1, 1), W.single_conv(1, 17, 13, 11, 40, 5, 1, 2), W.single_conv(3, 90, 7, 9, 33, 1),
    W.straight_generic(2, 24, 17, 19, 40, 3, 1, 1, 48, 3, 1, 1), W.straight_generic(1, 24, 17, 19, 40, 1, 0, 1, 48, 1, 0, 1),
    W.straight_generic(1, 40, 14, 15, 16, 1, 0, 1, 32, 5, 2, 1), W.config(4, n=1, hw=17, c=40), W.config(3, n=1, hw=19, cin=48),
    W.split_fire_pool(n=1, cin=32, hw=15, s=16, e=64), W.merge_two_producers(1, c=24, h=9, w=11, cmid=40, cout=20),
    W.conv_gap_generic(2, 40, 9, 9, 70, 1, 0, 1), W.depthwise_pointwise(1, 18, 13, 9, 40),
    W.conv_pool_generic(1, 24, 19, 23, 40, 3, 1, 1, 3, 2, 1),
]


def named(wl, name):
    wl.name = name
    return wl


def pointwise_residual(k2):
    """Merge block whose first layer is 1x1."""
    b = W._Builder(f"residual_1_{k2}", 2, 24, 15, 14)
    t = b.conv(0, 40, 1, bn=True, relu=True, name="conv1")
    t = b.conv(t, 24, k2, pad=k2 // 2, bn=True, relu=False, name="conv2")
    b.add(t, 0, relu=True, name="add")
    b.group("merge", 0)
    return b.done(len(b.shapes) - 1, "relu_normal", 31)


# ... with these every kernel on three parts is a candidate of some block (test_abi_and_planner.py counts them)
WORKLOADS += [
    W.single_conv(2, 17, 13, 7, 52, 3, 1, 1), W.single_conv(1, 26, 6, 15, 20, 5, 1, 2),
    W.conv_pool_generic(1, 11, 10, 10, 20, 1, 0, 1, 3, 2, 1), W.depthwise_pointwise(1, 22, 11, 11, 16, k2=3, p2=1),
    W.straight_generic(2, 14, 12, 9, 12, 3, 1, 1, 32, 3, 1, 1), W.straight_generic(1, 12, 9, 18, 10, 1, 0, 1, 25, 3, 1, 1),
    W.straight_generic(1, 48, 34, 27, 8, 1, 0, 1, 23, 5, 2, 1), W.straight_generic(1, 9, 15, 11, 9, 3, 1, 1, 22, 5, 2, 1),
    W.straight_generic(1, 35, 8, 41, 13, 3, 1, 1, 80, 1, 0, 1), pointwise_residual(3), pointwise_residual(1),
    named(W.config(4, n=1, c=21, hw=9), "residual_21x9"),
    named(W.split_fire_pool(n=1, cin=23, hw=10, s=16, e=48), "firepool_23x10"),
    named(W.config(3, n=1, cin=419, hw=10, s=48, e=128), "fire_419x10"), named(W.config(3, n=2, cin=336, hw=18, s=48, e=48), "fire_336x18"),
    named(W.config(3, n=1, cin=32, hw=10, s=16, e=48), "fire_32x10"),
    # strides in either layer, and paddings beyond half of the filter
    W.single_conv(2, 40, 19, 23, 70, 3, 2, 1), W.single_conv(1, 20, 17, 14, 33, 5, 3, 4),
    named(W.straight_generic(2, 24, 17, 19, 40, 3, 1, 2, 48, 3, 1, 1), "straight_s2_s1"),
    named(W.straight_generic(2, 24, 19, 21, 40, 3, 2, 1, 48, 3, 0, 2), "straight_s1_s2"),
    named(W.straight_generic(2, 40, 19, 21, 16, 1, 0, 1, 32, 5, 3, 2), "straight_1x1_5x5_s2"),
    named(W.conv_pool_generic(1, 24, 29, 23, 40, 3, 1, 2, 2, 2, 0), "convpool_s2"),
    named(W.depthwise_pointwise(2, 18, 23, 19, 40, s2=2), "dwpw_s2"),
]
OPTIONS = {"fire_32x10": {"force_tile_h": 10, "force_tile_w": 8}}


def run_candidates(wl, x, params):
    """{variant: output} of the fused launch, one candidate per variant, and the fp32 variants' ids first."""
    from paper_2007_06000_amd.session import Session
    s = Session(wl, x, params, **OPTIONS.get(wl.name, {}))
    out = {}
    for c in range(s.plan.num_candidates(True, 0)):
        v = s.plan.candidate_info(True, 0, c)["variant"]
        if v in out:
            continue
        s.plan.select_candidate(True, 0, c)
        print(f"[case] {wl.name} variant {v} candidate {c}", flush=True)
        out[v] = s.output(True)
    fp32 = {v: y for v, y in out.items() if v < FIRST}
    split = {v: y for v, y in out.items() if FIRST <= v < END}
    assert fp32 and split, sorted(out)
    return fp32, split


@pytest.mark.parametrize("wl", WORKLOADS, ids=lambda w: w.name)
def test_error_is_no_larger_than_with_fp32_operations(wl):
    # The reference is float64 with one rounding per layer output: both kernels share those roundings (2^-24 per element
    # and layer), hence the floor below which neither is told apart.
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params).astype(np.float64)
    fp32, split = run_candidates(wl, x, params)

    def err(y):
        return np.linalg.norm(y.astype(np.float64) - ref) / np.linalg.norm(ref)
    worst = max(err(y) for y in fp32.values())
    for v, y in split.items():
        assert err(y) <= max(worst, 2.0 ** -23), (v, err(y), worst)
    # Not only than the worst of them.  The fp32 kernels differ in the order of their sums alone; over 200 or more outputs the
    # norm varies by about 1 / sqrt(200) = 7 % between orders, so that the best is the same error up to three times that.
    best = min(err(y) for y in fp32.values())
    for v, y in split.items():
        assert err(y) <= max(1.25 * best, 2.0 ** -23), (v, err(y), best)


@pytest.mark.parametrize("special", [np.inf, -np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("wl", WORKLOADS, ids=lambda w: w.name)
def test_values_without_bf16_parts(wl, special):
    # one such value: whatever it reaches is what the fp32 kernels make of it, everything else is untouched
    x, params = W.make_tensors(wl)
    x[0, 1, x.shape[2] // 2, x.shape[3] // 2] = special
    fp32, split = run_candidates(wl, x, params)
    ref = next(iter(fp32.values()))
    fin = np.isfinite(ref)
    assert fin.any() or wl.name.startswith("convgap")
    for v, y in split.items():
        assert (np.isnan(y) == np.isnan(ref)).all(), v
        assert (np.isposinf(y) == np.isposinf(ref)).all() and (np.isneginf(y) == np.isneginf(ref)).all(), v
        a, b = y[fin].astype(np.float64), ref[fin].astype(np.float64)
        d, reached = np.abs(a - b), np.maximum(np.abs(a), np.abs(b)) > 1e20
        assert (d <= 1e-4 + 1e-4 * np.abs(b))[~reached].all(), (v, d[~reached].max())
        # sums that hold 3.4e38 * w: up to a few hundred roundings of 2^-24 of that magnitude
        assert (d[reached] <= 2.0 ** -16 * 3.4e38).all(), (v, d[reached].max())


@pytest.mark.parametrize("special", [np.inf, 3.4e38])
@pytest.mark.parametrize("wl", WORKLOADS, ids=lambda w: w.name)
def test_a_filter_value_without_bf16_parts_in_each_layer(wl, special):
    for layer in [i for i, ly in enumerate(wl.layers) if ly.op == "conv"]:
        x, params = W.make_tensors(wl)
        w = params[layer]["w"]
        w[3, min(5, w.shape[1] - 1), w.shape[2] // 2, w.shape[3] // 2] = special
        fp32, split = run_candidates(wl, x, params)
        ref = next(iter(fp32.values()))
        # what it does not reach is untouched
        fin = np.isfinite(ref) & (np.abs(ref) < 1e20)
        for v, y in split.items():
            assert (np.isfinite(y) == np.isfinite(ref)).all() and (np.isnan(y) == np.isnan(ref)).all(), (layer, v)
            assert (np.abs(y[fin] - ref[fin]) <= 1e-4 + 1e-4 * np.abs(ref[fin])).all(), (layer, v)


@pytest.mark.parametrize("special", [np.inf, 3.4e38])
def test_filters_without_bf16_parts(special):
    wl = W.config(4, n=1, hw=17, c=40)
    x, params = W.make_tensors(wl)
    params[2 if 2 in params else 1]["w"][3, 5, 1, 1] = special
    fp32, split = run_candidates(wl, x, params)
    ref = next(iter(fp32.values()))
    for v, y in split.items():
        assert (np.isfinite(y) == np.isfinite(ref)).all() and (np.isnan(y) == np.isnan(ref)).all(), v


@pytest.mark.parametrize("wl", WORKLOADS, ids=lambda w: w.name)
def test_products_just_below_the_largest_float(wl):
    # (2 - 2^-9)^2 * 2^126 is below FLT_MAX, while the product of the factors rounded to bf16 is 2^128: one pixel and one
    # filter value of the first layer, so that one of its sums is within 2^-8 of FLT_MAX.
    big = np.float32(2.0 - 2.0 ** -9) * np.float32(2.0 ** 63)
    x, params = W.make_tensors(wl)
    x[0, 1, x.shape[2] // 2, x.shape[3] // 2] = big
    first = wl.layers[0]
    w = params[0]["w"]
    k = first.k // 2
    w[0, 1 if first.groups == 1 else 0, k, k] = big
    if first.groups != 1:
        x[0, 0, x.shape[2] // 2, x.shape[3] // 2] = big
    if params[0]["scale"] is not None:
        params[0]["scale"][0] = 1.0
    fp32, split = run_candidates(wl, x, params)
    ref = next(iter(fp32.values()))
    assert all((np.isfinite(y) == np.isfinite(ref)).all() for y in fp32.values())
    for v, y in split.items():
        assert (np.isfinite(y) == np.isfinite(ref)).all(), v
        fin = np.isfinite(ref)
        # sums that hold a term near FLT_MAX: up to a few hundred roundings of 2^-24 of that magnitude
        d = np.abs(y[fin].astype(np.float64) - ref[fin].astype(np.float64))
        reached = np.abs(ref[fin]) > 1e10
        assert (d <= 1e-4 + 1e-4 * np.abs(ref[fin]))[~reached].all(), (v, d[~reached].max())
        assert (d <= 2.0 ** -16 * 3.4e38)[reached].all(), (v, d[reached].max())


@pytest.mark.parametrize("wl", [w for w in WORKLOADS if len([ly for ly in w.layers if ly.op == "conv"]) > 1], ids=lambda w: w.name)
def test_passes_repeat_bit_for_bit_around_an_infinite_intermediate(wl):
    # one sum of the first layer overflows: what a wave then does must not depend on how far the others are
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    # (the input pixel under the centre tap of an even position of the intermediate, which a strided second layer reads too)
    first = wl.layers[0]
    k = first.k // 2
    y0, x0 = [wl.shapes[first.out][d] // 4 * 2 * first.stride - first.pad + k for d in (2, 3)]
    x[0, 0, y0, x0] = 3e38
    params[0]["w"][0, 0, k, k] = 4.0
    s = Session(wl, x, params, **OPTIONS.get(wl.name, {}))
    seen = set()
    for c in range(s.plan.num_candidates(True, 0)):
        v = s.plan.candidate_info(True, 0, c)["variant"]
        if v < FIRST or v in seen:
            continue
        seen.add(v)
        s.plan.select_candidate(True, 0, c)
        print(f"[case] {wl.name} variant {v} candidate {c}", flush=True)
        first = s.output(True)
        assert not np.isfinite(first).all(), v
        for _ in range(10):
            assert s.output(True).tobytes() == first.tobytes(), v
    assert seen


@pytest.mark.parametrize("where", ["input", "filter 1", "filter 2"])
@pytest.mark.parametrize("wl", WORKLOADS, ids=lambda w: w.name)
def test_error_on_small_operands_is_no_larger_than_with_fp32_operations(wl, where):
    # Values around 2^-118 have bits below 2^-133, the smallest bf16 number; the other operand is scaled up so that the
    # results are ordinary floats.  ("filter 2" makes the filters of the later layers small and the intermediate large.)
    x, params = W.make_tensors(wl)
    convs = [i for i, ly in enumerate(wl.layers) if ly.op == "conv"]
    small, large = np.float32(2.0 ** -118), np.float32(2.0 ** 60)
    if where == "filter 2" and len(convs) == 1:
        pytest.skip("one layer")
    x *= small if where == "input" else large
    for i in convs:
        first = wl.layers[i].inputs[0] == wl.input_id
        if where == "filter 1" and first or where == "filter 2" and not first:
            params[i]["w"] *= small
        if params[i]["shift"] is not None:
            params[i]["shift"] *= np.float32(0.0)
    if where == "input":
        for i in convs[-1:]:
            params[i]["w"] *= large
    ref = xlo.forward(wl, x, params).astype(np.float64)
    fp32, split = run_candidates(wl, x, params)

    def err(y):
        scale = np.abs(ref).max()
        return float(np.linalg.norm(y / scale - ref / scale) / np.linalg.norm(ref / scale))
    # The same fp32 operations with the K steps in another order: as many roundings, other ones.  The norm over the 200 or
    # more outputs of a case varies by about 1 / sqrt(200) = 7 % between orders; 25 % is more than three times that.
    worst = max(err(y) for y in fp32.values())
    for v, y in split.items():
        assert err(y) <= max(1.25 * worst, 2.0 ** -23), (v, err(y), worst)
