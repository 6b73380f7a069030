"""bench.py's line on stdout: complete in what names the run and its figures, and short."""
import json

import pytest

import bench


def record(launches=30, blocks=15):
    row = {"layers": "fire2_squeeze..fire2_expand3x3", "us": 46.123456789, "frac": 0.71234567891, "adopted": [{"variant": 461}] * 12}
    block = dict(row, workload="table1_c1_batch1:merge2_64x56x56_256_64", wall_ms_fused=0.1, batch=32, ms_fused=0.123456789, images_per_s=123456.789012,
                 speedup_vs_unfused=1.23456789, bound="per launch", slowest5=[[1.2, 3]] * 5)
    return {"metric": "images/sec", "value": 113456.78901234, "unit": "images/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 0.5641234,
            "config": {"workload": "cfg5", "batch": 64, "blocks_run_layer_by_layer": ["fire6_squeeze1x1"] * 6, "tiles": "xl_tune " * 4},
            "roofline": {"bound": "mfma", "achieved": 118.253717, "frac": 0.75177187, "kernel": "conv10..gap", "traffic": None, "launch": 11},
            "per_launch": [row] * launches, "per_launch_note": "x" * 300, "target_60pct": {"met_by": ["y"] * launches},
            "peaks": {"published": {}, "measured": {"copy_gbs": 5312.123456, "mfma_f32_tflops": 151.123456}, "how": "z" * 200},
            "blocks": [dict(block, workload=f"{i}_" + block["workload"]) for i in range(blocks)] + [{"workload": "table1_a1", "error": "OSError()"}],
            "bf16x3": {"value": 1.5e5, "roofline": {"frac": 0.5}, "per_launch": [row] * launches, "blocks": [dict(block, workload=f"cfg{i}") for i in range(3)]},
            "cpu_baseline": {"value": 55.5, "unit": "images/s", "cores": 16, "kind": "oracle", "sample": "w" * 100}}


def test_the_line_is_short_and_keeps_the_figures():
    out = record()
    line = bench.short_line(out)
    assert len(json.dumps(line)) < 4000
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "config", "cpu_baseline"):
        assert line[key] == out[key]
    assert abs(line["roofline"]["frac"] - out["roofline"]["frac"]) < 1e-4 and line["measured_peaks"]["copy_gbs"] > 5000
    assert len(line["blocks"]) == len(out["blocks"]) and line["blocks"]["table1_a1"] == "OSError()"
    assert line["blocks"]["0_table1_c1_batch1"] == [32, 0.12346, 1.2346, 0.71235]
    assert line["bf16x3"]["value"] == 1.5e5 and len(line["bf16x3"]["blocks"]) == 3


def test_the_line_of_a_run_without_the_extra_rows():
    out = record()
    for key in ("blocks", "bf16x3", "cpu_baseline"):
        del out[key]
    assert bench.short_line(out)["value"] == out["value"]


def test_saved_candidates_are_taken_only_where_they_are_what_they_were():
    import xl_workloads as W
    from paper_2007_06000_amd import binding as B
    p = B.Plan(W.config(4))
    saved = {"layer_by_layer_blocks": [], "candidates": [[1, 0, 3, bench.configuration(p, True, 0, 3)], [0, 1, 2, bench.configuration(p, False, 1, 2)]]}
    bench.apply_candidates(p, saved)
    assert (p.candidate_info(True, 0)["candidate"], p.candidate_info(False, 1)["candidate"]) == (3, 2)
    # a list in another order, and one without the candidate
    first = saved["candidates"][0]
    for place in (4, 64):
        with pytest.raises(SystemExit):
            bench.apply_candidates(p, dict(saved, candidates=[first[:2] + [place, first[3]]]))
    bench.apply_candidates(p, dict(saved, candidates=[[1, 0, 5]]))
    assert p.candidate_info(True, 0)["candidate"] == 5
