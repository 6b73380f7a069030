"""The stem on the bf16 matrix cores (variant 170): image widths that end inside a wave's 31 pixels and inside a 16-byte
piece, heights that end inside a wave's rows, output channels that fill no row tile, and values without bf16 parts."""
import numpy as np
import pytest

import xl_workloads as W
from oracle import xlo


def stem(n, h, w, c, **kw):
    return W.conv_pool_generic(n, 3, h, w, c, 3, 0, 2, 3, 2, 0, **kw)


CASES = [stem(2, 64, 64, 64), stem(1, 7, 7, 16), stem(1, 9, 8, 33), stem(3, 11, 131, 20, relu=False), stem(2, 135, 133, 96, bn=True),
         stem(1, 63, 130, 70), stem(1, 40, 129, 64, relu=False, bn=True), stem(2, 30, 254, 8), stem(1, 256, 13, 32)]


def candidates(p):
    out = {}
    for c in range(p.num_candidates(True, 0)):
        v = p.candidate_info(True, 0, c)["variant"]
        if v == 170:
            out.setdefault(v, []).append(c)
    return out


def test_where_the_kernels_are_planned():
    from paper_2007_06000_amd import binding as B
    for precision in (0, 1):
        for wl in CASES:
            assert set(candidates(B.Plan(wl, precision=precision))) == {170}, wl.name
    for wl in (W.conv_pool_generic(1, 3, 64, 64, 32, 3, 1, 2, 3, 2, 0), W.conv_pool_generic(1, 4, 64, 64, 32, 3, 0, 2, 3, 2, 0),
               W.conv_pool_generic(1, 3, 64, 64, 32, 3, 0, 1, 3, 2, 0), W.conv_pool_generic(1, 3, 64, 64, 32, 3, 0, 2, 3, 2, 1)):
        assert not candidates(B.Plan(wl)), wl.name


@pytest.mark.parametrize("n,h,w,c", [(8, 224, 224, 64), (64, 224, 224, 64), (16, 150, 200, 96)])
def test_the_choice_where_the_chip_is_filled_in_either_precision(n, h, w, c):
    from paper_2007_06000_amd import binding as B
    for precision in (0, 1):
        p = B.Plan(stem(n, h, w, c), precision=precision)
        assert p.candidate_info(True, 0, 0)["variant"] == 170, precision
        # (two parts: the kernels on fp32 operations stay behind)
        costs = [(p.candidate_info(True, 0, i)["variant"] < 170, p.candidate_info(True, 0, i)["model_cost_us"]) for i in range(p.num_candidates(True, 0))]
        assert costs == (sorted(costs) if precision else sorted(costs, key=lambda t: t[1]))


@pytest.mark.parametrize("cout", [32, 64])
def test_a_fixed_number_of_workgroups_per_tile_is_kept(cout):
    from paper_2007_06000_amd import binding as B
    for split in (1, 2, 3):
        p = B.Plan(stem(8, 224, 224, cout), force_cout_split=split)
        mine = {p.candidate_info(True, 0, c)["cout_split"] for cs in candidates(p).values() for c in cs}
        assert mine == ({split} if split == cout // 32 else set()), split


@pytest.mark.gpu
@pytest.mark.parametrize("wl", CASES, ids=lambda w: w.name)
def test_against_the_oracle(wl):
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    s = Session(wl, x, params)
    for v, cs in candidates(s.plan).items():
        for c in cs:
            print(f"[case] {wl.name} {s.plan.candidate_info(True, 0, c)}", flush=True)
            s.plan.select_candidate(True, 0, c)
            y = s.output(True)
            # 28 terms and one rounding: 2^-21 is 8 roundings
            assert np.linalg.norm(y - ref) <= 2.0 ** -21 * np.linalg.norm(ref), (v, c)


def thin(s, variants=(130, 140)):
    """The result of a kernel on plain multiply-adds."""
    c = [c for c in range(s.plan.num_candidates(True, 0)) if s.plan.candidate_info(True, 0, c)["variant"] in variants][0]
    s.plan.select_candidate(True, 0, c)
    return s.output(True)


@pytest.mark.gpu
@pytest.mark.parametrize("special", [np.inf, -np.inf, np.nan, 3e38, 2.0 ** 100, 2.0 ** -120, 2.0 ** -140])
@pytest.mark.parametrize("wl", CASES[3:6], ids=lambda w: w.name)
def test_values_without_bf16_parts_and_large_ones(wl, special):
    """In the input, in a filter and in a shift: what plain multiply-adds make of them, and nothing else changes."""
    from paper_2007_06000_amd.session import Session
    for where in ("x", "w", "shift"):
        x, params = W.make_tensors(wl)
        value = np.float32(special * (1 + 2.0 ** -20 if abs(special) < 1 else 1))
        if where == "x" and np.isnan(special):
            x[0, 1, 2:11, 20:34] = value        # (pooling drops a NaN beside numbers: whole windows of them)
        elif where == "x":
            x[0, 1, 5, 20:24] = value
        elif where == "w":
            params[0]["w"][3, 1, 1, 2] = value
        else:
            params[0]["shift"][5] = value
        s = Session(wl, x, params)
        # (an activation makes 0 of a NaN in variant 130, and leaves it in 140, which has the stem's shape alone, and in the stem kernel)
        ref = thin(s, (140,) if np.isnan(special) else (130, 140))
        fin = np.isfinite(ref) & (np.abs(ref) < 1e20)
        assert np.isnan(ref).any() or not np.isnan(special)
        for v, cs in candidates(s.plan).items():
            s.plan.select_candidate(True, 0, cs[0])
            y = s.output(True)
            assert (np.isnan(y) == np.isnan(ref)).all(), (where, v)
            assert (np.isposinf(y) == np.isposinf(ref)).all() and (np.isneginf(y) == np.isneginf(ref)).all(), (where, v)
            assert (np.abs(y[fin] - ref[fin]) <= 1e-5 + 1e-5 * np.abs(ref[fin])).all(), (where, v)


@pytest.mark.gpu
def test_error_is_no_larger_than_with_multiply_adds():
    from paper_2007_06000_amd.session import Session
    wl = stem(2, 135, 133, 96, bn=True)
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params).astype(np.float64)
    s = Session(wl, x, params)
    err = lambda y: np.linalg.norm(y - ref) / np.linalg.norm(ref)
    plain = err(thin(s))
    for v, cs in candidates(s.plan).items():
        s.plan.select_candidate(True, 0, cs[0])
        assert err(s.output(True)) <= plain, v


@pytest.mark.gpu
@pytest.mark.parametrize("n,h,w,c,d", [(2, 31, 133, 20, 40), (3, 64, 64, 64, 33)])
def test_channel_slices_of_a_wider_tensor(n, h, w, c, d):
    from paper_2007_06000_amd.session import Session
    from test_gpu_chain import beside
    wl = beside([stem(n, h, w, c), stem(n, h, w, d, relu=False)], "stems_beside")
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    s = Session(wl, x, params)
    for k in range(8):
        for launch in range(2):
            mine = [i for i in range(s.plan.num_candidates(True, launch)) if s.plan.candidate_info(True, launch, i)["variant"] == 170]
            s.plan.select_candidate(True, launch, mine[k % len(mine)])
        y = s.output(True)
        for part in (slice(0, c), slice(c, None)):      # (28 terms and one rounding, as above)
            assert np.linalg.norm((y - ref)[:, part]) <= 2.0 ** -21 * np.linalg.norm(ref[:, part]), k
