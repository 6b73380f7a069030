"""Pointwise -> pointwise blocks with the intermediate in registers (variants 320 to 343 and 520 to 543): against the oracle at
partial tiles, pixels of several images in a wave, channels that fill neither K steps nor row tiles, and with the values
that have no bf16 parts."""
import numpy as np
import pytest

import test_gpu_split_operands as S
import xl_workloads as W
from oracle import xlo


def two(n, c, h, w, cmid, cout):
    return W.merge_two_producers(n, c=c, h=h, w=w, cmid=cmid, cout=cout)


def one(n, c, h, w, cmid, cout):
    return W.straight_generic(n, c, h, w, cmid, 1, 0, 1, cout, 1, 0, 1)


# every kernel: producers, K steps of layer 1, row tiles of layer 2, in the order of their ids
KERNELS = [(n1, nkg, nrt) for n1 in (1, 2) for nkg in range(1, 7 if n1 == 1 else 5) for nrt in ((1, 2, 3) if n1 == 1 and nkg <= 4 else (1, 2))]
# (workload, kernel): pixels that end inside a wave, waves of several images, channels that end inside K steps and row tiles
CASES = [
    (two(3, 16, 5, 7, 32, 16), (2, 1, 1)), (two(40, 9, 3, 3, 33, 40), (2, 1, 2)), (two(1, 24, 64, 65, 16, 20), (2, 2, 1)),
    (two(33, 30, 2, 3, 100, 64), (2, 2, 2)), (two(2, 37, 9, 9, 50, 31), (2, 3, 1)), (two(5, 40, 11, 13, 70, 64), (2, 3, 2)),
    (two(2, 64, 14, 14, 256, 32), (2, 4, 1)), (two(70, 63, 1, 1, 255, 64), (2, 4, 2)), (one(2, 8, 9, 9, 8, 8), (1, 1, 1)),
    (one(3, 16, 30, 31, 64, 64), (1, 1, 2)), (one(1, 13, 17, 16, 40, 96), (1, 1, 3)), (one(2, 17, 12, 9, 31, 32), (1, 2, 1)),
    (one(33, 30, 2, 3, 100, 64), (1, 2, 2)), (one(1, 32, 20, 20, 64, 65), (1, 2, 3)), (one(4, 48, 7, 7, 24, 20), (1, 3, 1)),
    (one(2, 45, 15, 15, 60, 50), (1, 3, 2)), (one(3, 40, 8, 9, 48, 96), (1, 3, 3)), (one(1, 64, 16, 16, 31, 31), (1, 4, 1)),
    (one(2, 50, 14, 13, 64, 33), (1, 4, 2)), (one(3, 50, 8, 9, 48, 96), (1, 4, 3)), (one(1, 80, 23, 5, 33, 10), (1, 5, 1)),
    (one(2, 70, 10, 10, 64, 64), (1, 5, 2)), (one(2, 90, 9, 9, 17, 20), (1, 6, 1)), (one(1, 96, 13, 31, 64, 64), (1, 6, 2)),
]
CASES = [(wl, KERNELS.index(k)) for wl, k in CASES]


def test_every_kernel_is_planned():
    from paper_2007_06000_amd import binding as B
    for precision, base in ((0, 520), (1, 320)):
        seen = set()
        for wl, k in CASES:
            p = B.Plan(wl, precision=precision)
            ids = {p.candidate_info(True, 0, c)["variant"] for c in range(p.num_candidates(True, 0))}
            assert base + k in ids, (wl.name, ids)
            seen.add(k)
        assert seen == set(range(len(KERNELS)))


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("wl,k", CASES, ids=lambda a: getattr(a, "name", ""))
def test_against_the_oracle(wl, k, precision):
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    bad = x.copy()
    bad[-1, -1, -1, -1] = np.inf        # stays at its pixel
    clean, broken = Session(wl, x, params, precision=precision), Session(wl, bad, params)
    want = (320 if precision else 520) + k
    done = 0
    for c in range(clean.plan.num_candidates(True, 0)):
        if clean.plan.candidate_info(True, 0, c)["variant"] != want:
            continue
        print(f"[case] {wl.name} variant {want} candidate {c}", flush=True)
        clean.plan.select_candidate(True, 0, c)
        y = clean.output(True)
        # three parts: sums of at most 256 terms and two roundings per layer, 2^-20 is 16 of them; two parts: 3 * 2^-16 of
        # the absolute sums at most, here within four times that of the result's norm
        assert np.linalg.norm(y - ref) <= (2.0 ** -12 if precision else 2.0 ** -20) * np.linalg.norm(ref)
        done += 1
    if not precision:
        for c in range(broken.plan.num_candidates(True, 0)):
            if broken.plan.candidate_info(True, 0, c)["variant"] == want:
                broken.plan.select_candidate(True, 0, c)
                z = broken.output(True)
                same = np.ones(z.shape, bool)
                same[-1, :, -1, -1] = False
                # (the other pixels of that wave are summed by fp32 operations: the same sums to a few roundings)
                assert np.linalg.norm((z - y)[same]) <= 2.0 ** -20 * np.linalg.norm(ref)
    assert done == 1


PARTS = [two(2, 24, 9, 11, 40, 20), two(1, 40, 7, 9, 70, 64), one(2, 90, 9, 9, 40, 20), one(1, 50, 13, 9, 48, 90)]


@pytest.mark.gpu
@pytest.mark.parametrize("special", [np.inf, -np.inf, np.nan, 3.4e38])
@pytest.mark.parametrize("wl", PARTS, ids=lambda w: w.name)
def test_values_without_bf16_parts(wl, special):
    S.test_values_without_bf16_parts(wl, special)
    if special in (np.inf, 3.4e38):
        S.test_a_filter_value_without_bf16_parts_in_each_layer(wl, special)


@pytest.mark.gpu
@pytest.mark.parametrize("wl", PARTS, ids=lambda w: w.name)
def test_errors_and_extremes(wl):
    S.test_error_is_no_larger_than_with_fp32_operations(wl)
    S.test_products_just_below_the_largest_float(wl)
    S.test_passes_repeat_bit_for_bit_around_an_infinite_intermediate(wl)
    for where in ("input", "filter 1", "filter 2"):
        S.test_error_on_small_operands_is_no_larger_than_with_fp32_operations(wl, where)


def first_candidates(s, wanted):
    """{variant: candidate} of the fused launch, the first of every variant that `wanted` takes."""
    out = {}
    for c in range(s.plan.num_candidates(True, 0)):
        v = s.plan.candidate_info(True, 0, c)["variant"]
        if wanted(v):
            out.setdefault(v, c)
    return out


def against_fp32_operations_on_two_parts(wl, x, params, base, count, what):
    """The kernels of a plan on two parts from id `base` on, against a kernel on fp32 operations of the same plan: the same infinities
    and NaN, and everything else within what two parts give."""
    from paper_2007_06000_amd.session import Session
    s = Session(wl, x, params, precision=1)
    s.plan.select_candidate(True, 0, min(first_candidates(s, lambda v: v < 200).values()))
    ref = s.output(True)
    fin = np.isfinite(ref)
    large = fin & (np.abs(ref) > 1e20)
    found = first_candidates(s, lambda v: base <= v < base + count)
    for v, c in found.items():
        print(f"[case] {wl.name} {what} variant {v} candidate {c}", flush=True)
        s.plan.select_candidate(True, 0, c)
        y = s.output(True)
        assert (np.isnan(y) == np.isnan(ref)).all() and (np.isposinf(y) == np.isposinf(ref)).all() and (np.isneginf(y) == np.isneginf(ref)).all(), (v, what)
        d = np.abs(np.where(fin, y, 0).astype(np.float64) - np.where(fin, ref, 0).astype(np.float64))
        # 3 * 2^-16 of the absolute sums of the last layer at most: at the scale of these blocks the library's bar, and where a
        # large value is part of the sums (up to 256 terms of random sign, their absolute sum within four times the largest
        # result) 2^-12 of the largest
        assert (d <= 1e-4 + 1e-4 * np.abs(ref))[fin & ~large].all(), (v, what, d[fin & ~large].max())
        assert not large.any() or d[large].max() <= 2.0 ** -12 * np.abs(ref[large]).max(), (v, what)
    return set(found)


@pytest.mark.gpu
@pytest.mark.parametrize("special", [np.inf, -np.inf, np.nan, 3.4e38, 2.0 ** -134])
@pytest.mark.parametrize("wl,k", CASES, ids=lambda a: getattr(a, "name", ""))
def test_values_without_bf16_parts_on_two_parts(wl, k, special):
    """Layer 1 takes three parts there too, and the whole operands of the wave that starts again are filters of two in layer 2: such a
    value in the input and in the filter of every layer 1."""
    value = np.float32(special) * np.float32(1 + 2.0 ** -10 if special == 2.0 ** -134 else 1)
    for where in [None] + [i for i, ly in enumerate(wl.layers) if ly.op == "conv" and ly.inputs[0] == wl.input_id]:
        x, params = W.make_tensors(wl)
        if where is None:
            x[0, 1, x.shape[2] // 2, x.shape[3] // 2] = value
        else:
            params[where]["w"][3, 5, 0, 0] = value
            if params[where]["scale"] is not None:
                params[where]["scale"][3] = 1.0
        assert against_fp32_operations_on_two_parts(wl, x, params, 320, len(KERNELS), f"{special} in {where}") >= {320 + k}


def beside(blocks, name):
    """Blocks on one input, their results next to each other in one tensor."""
    n, c, h, w = blocks[0].shapes[0]
    b = W._Builder(name, n, c, h, w)
    t = None
    for wl in blocks:
        first, of = len(b.layers), {0: 0}
        for ly in wl.layers:
            ins = [of[i] for i in ly.inputs]
            of[ly.out] = (b.conv(ins[0], ly.cout, ly.k, ly.stride, ly.pad, bias=ly.bias, bn=ly.bn, relu=ly.relu, name=ly.name) if ly.op == "conv"
                          else b.maxpool(ins[0], ly.k, ly.stride, ly.pad) if ly.op == "maxpool" else b.add(*ins, relu=ly.relu))
        b.group(wl.groups[0].mode, first)
        t = of[wl.output_id] if t is None else b.concat(t, of[wl.output_id])
    return b.done(t, blocks[0].input_dist, 41)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("blocks", [[one(2, 40, 9, 11, 48, 20), one(2, 40, 9, 11, 33, 70)], [two(3, 24, 7, 9, 40, 33), one(3, 24, 7, 9, 20, 31)],
                                    [one(1, 24, 13, 10, 16, 64), two(1, 24, 13, 10, 50, 17)]], ids=["one_one", "two_one", "one_two"])
def test_channel_slices_of_a_wider_tensor(blocks, precision):
    from paper_2007_06000_amd.session import Session
    wl = beside(blocks, "chains_beside")
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    s = Session(wl, x, params, precision=precision)
    base = 320 if precision else 520
    for launch in range(2):
        chain = [c for c in range(s.plan.num_candidates(True, launch)) if base <= s.plan.candidate_info(True, launch, c)["variant"] < base + len(KERNELS)]
        assert len(chain) == 1
        s.plan.select_candidate(True, launch, chain[0])
    y = s.output(True)
    first = blocks[0].shapes[blocks[0].output_id][1]
    for part in (slice(0, first), slice(first, None)):      # (bounds as in test_against_the_oracle)
        assert np.linalg.norm((y - ref)[:, part]) <= (2.0 ** -12 if precision else 2.0 ** -20) * np.linalg.norm(ref[:, part])
