"""Kernels whose first, pointwise layer reads memory (variants 370 to 384 and 570 to 584): channels that fill neither K steps of 32 nor
row tiles of 16, reductions in one piece, divided between waves and in chunks, strides, tiles over the image's edge, padded poolings."""
import numpy as np
import pytest

import xl_workloads as W
from oracle import xlo


def named(wl, name):
    wl.name = name
    return wl


# (workload, options): with these every kernel is a candidate, and the reduction of layer 1 divided by 1, 2, 4 and 8
CASES = [
    (named(W.config(3, n=1, hw=13, cin=512, s=64, e=256), "fire_512"), {}), (named(W.config(3, n=2, hw=9, cin=37, s=16, e=48), "fire_37"), {}),
    (named(W.config(3, n=1, hw=20, cin=130, s=48, e=96), "fire_130"), {}), (named(W.config(3, n=1, hw=5, cin=8, s=24, e=33), "fire_8"), {}),
    (named(W.config(3, n=2, hw=23, cin=65, s=9, e=70), "fire_65"), {"force_tile_h": 8, "force_tile_w": 23}),
    (named(W.config(3, n=1, hw=19, cin=97, s=31, e=64), "fire_97"), {"force_tile_h": 10, "force_tile_w": 19}),
    (named(W.config(3, n=1, hw=14, cin=600, s=64, e=64), "fire_600"), {"force_tile_h": 7, "force_tile_w": 7}),
    (named(W.config(3, n=1, hw=16, cin=33, s=50, e=64), "fire_33"), {}), (named(W.config(3, n=2, hw=9, cin=300, s=16, e=64), "fire_300"), {"force_tile_h": 2, "force_tile_w": 4}),
    (named(W.split_fire_pool(n=2, cin=64, hw=15, s=16, e=64), "firepool_64"), {}), (named(W.split_fire_pool(n=1, cin=200, hw=13, s=64, e=100, pp=1), "firepool_200"), {}),
    (named(W.split_fire_pool(n=1, cin=90, hw=19, s=48, e=64), "firepool_90"), {}), (named(W.split_fire_pool(n=3, cin=31, hw=12, s=32, e=64), "firepool_31"), {}),
    (named(W.straight_generic(1, 40, 19, 21, 16, 1, 0, 1, 32, 5, 3, 2), "conv5_40"), {}), (named(W.straight_generic(2, 130, 14, 15, 17, 1, 0, 2, 40, 5, 2, 1), "conv5_130"), {}),
]
CASES = [pytest.param(wl, o, id=wl.name) for wl, o in CASES]


def candidates(p, base):
    """{(variant, waves that divide layer 1): [candidate]}"""
    out = {}
    for c in range(p.num_candidates(True, 0)):
        i = p.candidate_info(True, 0, c)
        if base <= i["variant"] < base + 15:
            out.setdefault((i["variant"] - base, i["waves_cout_1"]), []).append(c)
    return out


def test_every_kernel_is_planned():
    from paper_2007_06000_amd import binding as B
    for precision, base in ((0, 570), (1, 370)):
        seen, kparts = set(), set()
        for case in CASES:
            wl, options = case.values
            got = candidates(B.Plan(wl, precision=precision, **options), base)
            assert got, wl.name
            seen |= {v for v, _ in got}
            kparts |= {k for _, k in got}
        assert seen == set(range(15)) and kparts == {1, 2, 4, 8}, (precision, set(range(15)) - seen, kparts)


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("wl,options", CASES)
def test_against_the_oracle(wl, options, precision):
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    s = Session(wl, x, params, precision=precision, **options)
    for v, cs in candidates(s.plan, 370 if precision else 570).items():
        for c in cs:
            print(f"[case] {wl.name} kernel {v} candidate {s.plan.candidate_info(True, 0, c)}", flush=True)
            s.plan.select_candidate(True, 0, c)
            y = s.output(True)
            # three parts: sums of up to 600 terms of random sign in up to nine pieces and two roundings per layer, 2^-21 is eight of
            # them and four times what was measured; two parts in layer 2 leave out up to 3 * 2^-16 of the absolute sums, of the result's norm 2^-17.6 was measured
            assert np.linalg.norm(y - ref) <= (3 * 2.0 ** -17 if precision else 2.0 ** -21) * np.linalg.norm(ref), (v, c)


@pytest.mark.gpu
@pytest.mark.parametrize("special", [np.inf, np.nan, 3.4e38, 2.0 ** -134])
@pytest.mark.parametrize("wl,options", CASES)
def test_values_without_bf16_parts(wl, options, special):
    """One such value, in the input and in layer 1's filter: what the fp32 kernels make of it, and nothing else changes.  The small one comes with
    others of 2^-118, whose bits below the smallest bf16 number (2^-133) show in every output."""
    from paper_2007_06000_amd.session import Session
    for where in ("x", "w"):
        x, params = W.make_tensors(wl)
        value = np.float32(special) * np.float32(1 + 2.0 ** -10 if special < 1 else 1)
        small, other = (x, params[0]["w"]) if where == "x" else (params[0]["w"], x)
        if special < 1:
            small *= np.float32(2.0 ** -118)
            other *= np.float32(2.0 ** 60)
            for p in params.values():
                p["shift"][:] = 0
        small[(0, 1, x.shape[2] // 2, x.shape[3] // 2) if where == "x" else (3, 5, 0, 0)] = value
        if special < 1:         # what sums of the parts alone are: further off than the bound below
            ref = xlo.forward(wl, x, params)
            whole = small.copy()
            small[:] = np.round(small * np.float32(2.0 ** 100) * np.float32(2.0 ** 33)) * np.float32(2.0 ** -33) * np.float32(2.0 ** -100)
            assert np.linalg.norm((xlo.forward(wl, x, params) - ref) * 2.0 ** 58) > 2.0 ** -19 * np.linalg.norm(ref * 2.0 ** 58)
            small[:] = whole
        s = Session(wl, x, params, **options)
        fp32 = [c for c in range(s.plan.num_candidates(True, 0)) if s.plan.candidate_info(True, 0, c)["variant"] < 200][0]
        s.plan.select_candidate(True, 0, fp32)
        ref = s.output(True)
        fin = np.isfinite(ref) & (np.abs(ref) < 1e20)
        for v, cs in candidates(s.plan, 570).items():
            print(f"[case] {wl.name} {special} in {where} kernel {v} candidate {s.plan.candidate_info(True, 0, cs[0])}", flush=True)
            s.plan.select_candidate(True, 0, cs[0])
            y = s.output(True)
            assert (np.isnan(y) == np.isnan(ref)).all() and (np.isfinite(y) == np.isfinite(ref)).all(), (where, v)
            if special < 1:
                assert np.linalg.norm((y - ref) * 2.0 ** 58) <= 2.0 ** -20 * np.linalg.norm(ref * 2.0 ** 58), (where, v)
            else:
                assert (np.abs(y[fin] - ref[fin]) <= 1e-4 + 1e-4 * np.abs(ref[fin])).all(), (where, v)


FEW = [named(W.config(3, n=2, hw=9, cin=c, s=16, e=64), f"fire_{c}") for c in (1, 3, 7, 33)]
FEW += [named(W.split_fire_pool(n=2, cin=c, hw=11, s=24, e=64), f"firepool_{c}") for c in (1, 7, 39)] + [named(W.straight_generic(2, 3, 9, 9, 16, 1, 0, 1, 32, 5, 2, 1), "conv5_3")]


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("special", [np.inf, np.nan])
@pytest.mark.parametrize("wl", [pytest.param(wl, id=wl.name) for wl in FEW])
def test_channels_past_the_last_one_are_not_those_of_the_next_image(wl, special, precision):
    """Filters hold zeros for them, which only a finite value meets without harm: the second image has none."""
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    x[1] = special
    s = Session(wl, x, params, precision=precision)
    found = candidates(s.plan, 370 if precision else 570)
    assert found
    for v, cs in found.items():
        for c in cs:
            print(f"[case] {wl.name} kernel {v} candidate {s.plan.candidate_info(True, 0, c)}", flush=True)
            s.plan.select_candidate(True, 0, c)
            y = s.output(True)
            assert np.linalg.norm(y[0] - ref[0]) <= (2.0 ** -12 if precision else 2.0 ** -20) * np.linalg.norm(ref[0]), (v, c)


@pytest.mark.parametrize("wl,precision,slower", [
    (W.config(3, n=16, cin=96, hw=55, s=16, e=64), 0, 574),          # 19.2 us either way when warm, 20.8 and 20.4 in a program's first passes
    (W.config(3, n=64, cin=64, hw=54, s=16, e=64), 1, 374),          # 38.3 us, 33.1 of the kernel of two tiles
    (W.config(3, n=64, cin=96, hw=55, s=16, e=64), 1, 374),          # 49.9 us, 40.1
    (W.split_fire_pool(n=1, cin=256, hw=27, s=32, e=128), 1, 378),   # 12.7 us, 11.6 of the kernel that divides both layers
])
def test_the_first_choice_is_not_one_that_measured_slower(wl, precision, slower):
    from paper_2007_06000_amd import binding as B
    assert B.Plan(wl, precision=precision).candidate_info(True, 0, 0)["variant"] != slower
