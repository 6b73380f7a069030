"""Depthwise -> pointwise blocks wave by wave (variants 161 to 168) against the oracle, at partial tiles, partial channel
groups, one-pixel-wide images, paddings 0 to 3 and several cout tiles."""
import numpy as np
import pytest

import xl_workloads as W
from oracle import xlo

pytestmark = pytest.mark.gpu

IDS = range(161, 169)


@pytest.mark.parametrize("wl,expected", [
    (W.depthwise_pointwise(64, 13, 33, 47, 40), {161, 162, 165, 167}),
    (W.depthwise_pointwise(64, 6, 35, 33, 5), {161, 162, 164, 165}),
    (W.depthwise_pointwise(24, 16, 50, 50, 16, p1=0, relu1=False, bn2=True), {164, 165}),
    (W.depthwise_pointwise(300, 3, 17, 1, 5, bn1=True), {161, 162, 164, 165}),
    (W.depthwise_pointwise(64, 16, 66, 67, 30, s1=2), set()),
    (W.depthwise_pointwise(64, 13, 33, 30, 24, p1=2), {161, 162, 164, 165}), (W.depthwise_pointwise(64, 6, 35, 33, 40, p1=3), {161, 162, 165, 167}),
    (W.depthwise_pointwise(24, 16, 66, 67, 64), {161, 162, 165, 167, 168}),
    (W.depthwise_pointwise(24, 13, 33, 47, 70), {161, 162, 165, 167, 168}),
], ids=lambda a: getattr(a, "name", ""))
def test_against_the_oracle(wl, expected):
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    # a value that is not finite stays in its image: the neighbours' windows do not see it, whatever their padding reads
    bad = x.copy()
    bad[1, -1, -1, -1], bad[1, 0, 0, 0] = np.inf, np.nan
    clean, broken = Session(wl, x, params), Session(wl, bad, params)
    seen = set()
    for c in range(clean.plan.num_candidates(True, 0)):
        v = clean.plan.candidate_info(True, 0, c)["variant"]
        if v not in IDS or v in seen:
            continue
        seen.add(v)
        print(f"[case] {wl.name} variant {v} candidate {c}", flush=True)
        clean.plan.select_candidate(True, 0, c)
        broken.plan.select_candidate(True, 0, c)
        y, z = clean.output(True), broken.output(True)
        # 9 + cin fp32 multiply-adds per output in another order: a few roundings of 2^-24 in the norm
        assert np.linalg.norm(y - ref) <= 2.0 ** -20 * np.linalg.norm(ref), v
        others = [i for i in range(x.shape[0]) if i != 1]
        assert (y[others] == z[others]).all() and not np.isfinite(z[1]).all(), v
    assert seen >= expected and (expected or not seen), seen


@pytest.mark.parametrize("wl,tune", [
    (W.depthwise_pointwise(32, 16, 80, 80, 16, s2=2), False), (W.depthwise_pointwise(24, 13, 41, 50, 24, s2=3), False),
    (W.depthwise_pointwise(64, 8, 100, 100, 24, s2=2), True), (W.depthwise_pointwise(24, 13, 41, 50, 24, s2=3), True),
], ids=lambda a: getattr(a, "name", str(a)))
def test_a_strided_second_layer_runs_on_the_general_kernel(wl, tune):
    from paper_2007_06000_amd.session import Session
    x, params = W.make_tensors(wl)
    ref = xlo.forward(wl, x, params)
    s = Session(wl, x, params, tune=tune)
    assert np.linalg.norm(s.output(True) - ref) <= 2.0 ** -20 * np.linalg.norm(ref)
    seen = set()
    for c in range(s.plan.num_candidates(True, 0)):
        v = s.plan.candidate_info(True, 0, c)["variant"]
        if v not in seen:
            seen.add(v)
            print(f"[case] {wl.name} variant {v} candidate {c}", flush=True)
            s.plan.select_candidate(True, 0, c)
            assert np.linalg.norm(s.output(True) - ref) <= 2.0 ** -20 * np.linalg.norm(ref), v
