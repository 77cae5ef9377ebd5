"""bench.py's command-line contract: one JSON line with the agreed keys, and a clear refusal
of more than one GPU."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_more_than_one_gpu_is_refused_with_a_message():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert p.returncode != 0
    assert "one GPU" in (p.stderr + p.stdout)
    assert not p.stdout.strip().startswith("{")


def test_no_alu_fraction_without_a_count_and_no_counters_of_another_kernel():
    """k_dp_bound's scans are not counted, so it is not priced as if it scanned every source; a
    profile entry counts only for the kernel it was taken of."""
    sys.path.insert(0, ROOT)
    import bench
    assert bench.ops_per_relaxation("k_dp_bound", "bp", 96) is None
    assert bench.ops_per_relaxation("k_dp_bound", "nobp", 96) is None
    assert bench.ops_per_relaxation("k_dp_wide", "bp", 96) == 15 / 8 + 24 / 96
    entry = {"kernel": "void k_dp_wide<unsigned char, 8, true, 2, 64>", "lds_bytes": 1.0}
    assert bench.profile_of("k_dp_wide", entry) == entry
    assert bench.profile_of("k_dp_bound", entry) == {} and bench.profile_of("k_dp_bound", None) == {}


def test_profiled_figures_are_brought_to_one_front():
    """The line's bytes and times are of a layer front; a launch of two kernels covers several."""
    sys.path.insert(0, ROOT)
    import bench
    prof = dict(kernel="k", calls=20, solves=10, avg_us=46.0, traffic_bytes=92.0, lds_bytes=None)
    assert bench.per_front("k_dp_small", prof, 24) == \
        (dict(prof, avg_us=2.0, traffic_bytes=4.0), 23.0)
    assert bench.per_front("k_dp_class_fronts", prof, 47) == \
        (dict(prof, avg_us=2.0, traffic_bytes=4.0), 23.0)
    assert bench.per_front("k_dp_push", prof, 24) == (prof, 1.0)
    assert bench.per_front("k_dp_small", {}, 24) == ({}, 23.0)
    assert prof["avg_us"] == 46.0


def test_counters_of_other_sources_are_not_used(tmp_path):
    """A kernel that was rewritten keeps its name; its old bytes and durations are not its own."""
    sys.path.insert(0, ROOT)
    import bench
    from paper_2504_21411_amd.profile_summary import kernel_sources_digest
    src = tmp_path / "csrc"
    src.mkdir()
    digests = []
    for text in ("int a; // one\n", "int  a; /* two\n */\n", "int b;\n"):
        (src / "k.hip").write_text(text)
        digests.append(kernel_sources_digest(str(src)))
    assert digests[0] == digests[1] != digests[2]          # comments and layout do not count
    path = tmp_path / "traffic.json"
    for sources, own, kept in ((None, None, []), (digests[2], None, []), (kernel_sources_digest(), None, ["a", "b"]),
                               (digests[2], kernel_sources_digest(), ["b"])):
        d = {"commit": "c", "entries": {"a": {"kernel": "k"}, "b": {"kernel": "k"}}}
        if sources:
            d["sources"] = sources
        if own:
            d["entries"]["b"]["sources"] = own
        path.write_text(json.dumps(d))
        got = bench.load_profiled(str(path))
        assert sorted(got["entries"]) == kept and got["commit"] == ("c" if kept else None)
    assert bench.load_profiled(str(tmp_path / "none.json")) == {}


@pytest.mark.gpu
def test_bench_reports_no_alu_fraction_for_the_bounded_kernel():
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--mode", "bp-general",
                        "--also=", "--also-configs=", "--no-cpu-baseline", "--steps", "2",
                        "--warmup", "1", "--min-warmup-seconds", "0"],
                       capture_output=True, text=True, timeout=600)
    assert p.returncode == 0, p.stderr[-2000:]
    d = json.loads(p.stdout)
    r = d["roofline"]
    assert r["kernel"] == "k_dp_bound" and r["alu_frac"] is None and r["bound"] == "hbm"
    assert r["ops_per_relaxation"] is None and d["executed_grelax_per_s"] is None
    assert 0 < r["frac"] <= 1.0 and 0 < r["frac_single_chain"] <= 1.0 and d["value"] > 0
    assert r["traffic_profiled_kernel"] is None or "k_dp_bound" in r["traffic_profiled_kernel"]


@pytest.mark.gpu
@pytest.mark.parametrize("config", [0, 1])
def test_bench_prints_one_json_line_with_the_contract_keys(config):
    p = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--config", str(config),
                        "--steps", "3", "--warmup", "1", "--min-warmup-seconds", "0"],
                       capture_output=True, text=True, timeout=600)
    assert p.returncode == 0, p.stderr[-2000:]
    lines = [ln for ln in p.stdout.splitlines() if ln.strip()]
    assert len(lines) == 1
    d = json.loads(lines[0])
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
              "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config",
              "roofline", "cpu_baseline"):
        assert k in d, k
    assert d["n_gpus"] == 1 and d["steps"] == 3 and d["warmup"] == 1
    assert d["higher_is_better"] is True and d["vs_baseline"] is None and d["data"] == "synthetic"
    assert d["dtype"] == "f32" and d["unit"] == "Grelax/s" and "workload" in d["config"]
    assert "model" not in d["config"]
    r = d["roofline"]
    for k in ("bound", "achieved", "peak", "unit", "frac", "traffic"):
        assert k in r, k
    assert r["bound"] in ("hbm", "alu") and abs(r["frac"] - r["achieved"] / r["peak"]) < 1e-9
    c = d["cpu_baseline"]
    assert c["kind"] == "oracle" and c["cores"] == 1 and c["value"] > 0 and c["sample"]
    if config == 1:      # 64 instances: the oracle is also timed on several cores side by side
        m = d["cpu_baseline_all_cores"]
        assert m["kind"] == "oracle" and 2 <= m["cores"] <= 16 and m["value"] > 0 and m["sample"]
    assert d["value"] > 0 and d["ms_per_step"] > 0
    # value = nominal relaxations of the step / wall time of the step
    assert abs(d["value"] - d["config"]["relaxations_per_step"] / d["ms_per_step"] / 1e6) \
        <= 1e-6 * d["value"]
    # every other configuration is timed beside the main workload, each with its own
    # latency and roofline block (vector ALU, HBM and, where profiled, LDS)
    others = d["other_configs"]
    assert sorted(int(o["workload"][len("configs["):].split("]")[0]) for o in others) == \
        sorted({0, 1, 2, 4} - {config})
    for o in others + [d]:
        assert o["ms_per_step"] > 0 and o["forward_ms"] > 0 and o["budget_curve_ms"] > 0
        r = o["roofline"]
        assert 0 < r["frac"] <= 1.0 and r["alu_frac"] > 0 and "hbm_frac" in r and "lds" in r
        assert "frac_is" in r and r["kernel"].startswith("k_dp_")
        if r["concurrent_launches"] > 1:
            assert 0 < r["frac_single_chain"] <= 1.0
        if r["lds"] is not None:
            assert r["lds"]["peak"] > 70 and 0 <= r["lds"]["frac"] <= 1.5
    assert 0 < d["executed_fraction"] <= 1.0 and d["executed_grelax_per_s"] > 0
    assert "general_r_grelax_per_s" in d and "traffic_commit" in d
    assert d["target_50pct_of_roofline_met"] in (True, False)
    assert d["pipeline_reduce_ms"] > 0            # configs[4]: the pipeline-aware outer reduction
