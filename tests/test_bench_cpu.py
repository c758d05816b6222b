"""Host-side checks of bench.py that need no GPU: the single-GPU contract, the fixed headline choices, and the
roofline arithmetic on a made-up timing."""
import os
import subprocess
import sys
import types

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused():
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert res.returncode == 2 and "single-GPU" in res.stderr and res.stdout.strip() == ""


def test_headline_is_the_largest_config_in_one_fixed_form():
    sys.path.insert(0, ROOT)
    import bench
    assert bench.HEADLINE_CONFIG == 5 and bench.CONFIG_TEXT[5].startswith("configs[4]")
    # one fixed form per configuration (never the best of several): one fused launch for the single-layer
    # configurations, one persistent launch per pass for the 53-layer stacks
    assert bench.HEADLINE_FORM == {1: "fused", 2: "fused", 3: "fused", 4: "fused", 5: "fused_chain"}
    assert all(f in bench.POLICY_TEXT for f in bench.HEADLINE_FORM.values())
    # a step of the fused policy lasts at least several milliseconds at the measured pass times
    measured_us = {1: 5.5, 2: 8.8, 3: 14.4, 4: 49.4, 5: 451.0}
    for cfg, passes in bench.PASSES_PER_STEP.items():
        assert passes * measured_us[cfg] >= 10e3


def test_roofline_arithmetic():
    sys.path.insert(0, ROOT)
    import bench
    # config-5-like numbers: 49 launches, HBM-bound
    wl = types.SimpleNamespace(cfg=5, flops=65394180096, bytes=723700736, launches={"fused": 49, "fused_chain": 1},
                               launch_work=[(65394180096 // 49, 723700736 // 49)] * 49)
    r = bench.roofline(wl, "fused", {"event_us_per_pass_median": 490.0})
    assert r["bound"] == "hbm" and r["launches_per_pass"] == 49
    assert abs(r["avg_launch_us"] - 10.0) < 1e-9
    assert abs(r["achieved"] - 723700736 / 49 / 10e-6 / 1e9) < 1e-6 and abs(r["frac"] - r["achieved"] / 8000.0) < 1e-12
    assert abs(r["bound_us_per_pass"] - 723700736 / 8e12 * 1e6) < 0.05      # every launch is HBM-bound here
    assert abs(r["frac_of_own_bound"] - r["bound_us_per_pass"] / 490.0) < 1e-12
    c = bench.roofline(wl, "fused_chain", {"event_us_per_pass_median": 700.0})
    assert c["launches_per_pass"] == 1 and abs(c["avg_launch_us"] - 700.0) < 1e-9 and c["kernel"] == "st_chain_kernel"
    # a compute-bound workload is priced against the MFMA peak of its dtype
    wm = types.SimpleNamespace(cfg=4, flops=10 ** 12, bytes=10 ** 8, launches={"fused": 1}, launch_work=[(10 ** 12, 10 ** 8)])
    m = bench.roofline(wm, "fused", {"event_us_per_pass_median": 1000.0})
    assert m["bound"] == "mfma" and m["unit"] == "TFLOP/s" and abs(m["achieved"] - 1000.0) < 1e-9 and m["peak"] == 2516.6


def test_printed_line_is_short_and_whole():
    """The one line keeps every contract field and stays below the length that readers of the output's end see whole, with
    every form, every configuration and the oracle legs in the record."""
    import json
    sys.path.insert(0, ROOT)
    import bench
    timing = {"ms_per_step": 1 / 3, "us_per_pass": 1000 / 3, "event_ms_per_step": {"median": 1 / 3, "p10": 1 / 3, "p90": 1 / 3},
              "event_us_per_pass_median": 1000 / 3, "timed_region_s": 1 / 3, "tflops": 1000 / 3}
    forms = ["fused_chain", "fused"] + bench.BASELINES
    extras = {f: dict(timing) for f in ["fused_chain2", "fused_groups2", "space_only_chains", "fused_staggered", "time_only_staggered",
                                        "space_only_staggered", "space_only_free", "fused_cold"] + list(bench.PIPELINED)}
    wl = types.SimpleNamespace(cfg=5, flops=65394180096, bytes=723700736, launches={"fused": 49, "fused_chain": 1}, launch_work=[(1, 1)] * 49)
    roof = bench.roofline(wl, "fused_chain", timing)
    head = {"flops": 65394180096, "algorithmic_bytes": 723700736, "plan_build_us": 33.3, "work_items": 21741, "passes_per_step": 40, "steps": 20,
            "headline_form": "fused_chain", "policies": {f: dict(timing) for f in forms}, "value_tflops": 1000 / 3, "pct_bf16_mfma_peak": 100 / 3,
            "speedup_vs_time_only": 10 / 3, "speedup_vs_space_only": 10 / 3, "time_only_form": "time_only_retuned", "space_only_form": "space_only_retuned",
            "roofline": roof, "rooflines": {"fused": roof, "fused_chain": roof}, "extras": extras}
    line = {"metric": "aggregate conv TFLOP/s (% bf16 MFMA peak) + speedup vs time-only/space-only", "value": 1000 / 3, "unit": "TFLOP/s", "n_gpus": 1,
            "steps": 20, "warmup": 5, "ms_per_step": 1 / 3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
            "config": {"workload": bench.CONFIG_TEXT[5], "policy": bench.POLICY_TEXT["fused_chain"], "form": "fused_chain", "tenants": 8,
                       "passes_per_step": 40, "us_per_pass": 1000 / 3, "flops_per_pass": 65394180096},
            "event_ms_per_step": timing["event_ms_per_step"], "timed_region_s": 1 / 3, "pct_bf16_mfma_peak": 100 / 3, "speedup_vs_time_only": 10 / 3,
            "speedup_vs_space_only": 10 / 3, "baseline_forms": {"time_only": "time_only_retuned", "space_only": "space_only_retuned"},
            "policies": head["policies"], "launch_floor_us": 1.5, "plan_build_us": 33.3, "work_items": 21741, "gpu_max_hw_queues": "4",
            "roofline": dict(roof, achievable={"hbm_copy_GBps": 4639.123456789, "mfma_bf16_TFLOPs": 2049.123456789, "mfma_f16_TFLOPs": 2045.123456789,
                                               "mfma_f32_TFLOPs": 152.123456789, "published": {"hbm_GBps": 8000.0, "mfma_bf16_TFLOPs": 2516.6, "mfma_f32_TFLOPs": 157.3}}),
            "paper_context": bench.PAPER_CONTEXT, "rooflines": head["rooflines"], "extras": extras,
            "cpu_baseline": {"unit": "TFLOP/s", "cores": 16, "kind": "oracle", "value": 0.0271234567, "sample": "x" * 200,
                             "end_to_end_drift": {"what": "x" * 200, "tenants": [{"tenant": t, "max_abs_err_over_max_abs_ref": t / 300, "rel_l2": t / 300} for t in range(8)]},
                             "whole_configs": {str(c): {leg: {"seconds": 1 / 3, "gflops": 100 / 3, "threads": 16} for leg in ("all_threads", "single_thread")} for c in (1, 2, 3, 4)}},
            "per_config": {**{str(c): head for c in (1, 2, 3, 5)}, "4": {"error": "y" * 5000}, "geomean_speedup_vs_time_only": 10 / 3, "geomean_speedup_vs_space_only": 10 / 3}}
    extras["fused_cold"] = {"error": "z" * 5000}
    out = bench.printed(line)
    text = json.dumps(out)
    assert len(text) <= bench.MAX_LINE <= 8000 and "\n" not in text, len(text)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config"):
        assert out[k] == line[k], k
    assert out["roofline"]["frac"] == float(f"{roof['frac']:.6g}") and out["cpu_baseline"]["end_to_end_drift"]["rel_l2"] == float(f"{7 / 300:.6g}")
    assert set(out["per_config"]) == set(line["per_config"]) and out["per_config"]["2"]["tflops"] == 333.333


def test_traffic_is_reported_only_for_the_code_it_was_counted_on(tmp_path):
    sys.path.insert(0, ROOT)
    import bench
    path = tmp_path / "traffic.txt"
    path.write_text(f"# comment\n5 fused 10 5 {bench.kernel_sources_id()}\n4 fused 10 5 0123456789ab\n3 fused 10 5\n")
    assert bench.measured_traffic(5, "fused", str(path)) == 15.0
    assert bench.measured_traffic(5, "fused_chain", str(path)) is None      # not counted
    assert bench.measured_traffic(4, "fused", str(path)) is None            # counted on other code
    assert bench.measured_traffic(3, "fused", str(path)) is None            # on nobody knows what
    assert bench.measured_traffic(5, "fused", str(tmp_path / "none")) is None
    before = bench.kernel_sources_id()
    assert before == bench.kernel_sources_id() and len(before) == 12
