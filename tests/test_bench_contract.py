"""The benchmark's command-line contract: one JSON line with the agreed keys; more than one GPU is
refused with a message (this build is one EP rank's share on one GPU)."""
import json
import os
import re
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_19654_amd", "csrc")


def run_bench(*args, timeout=300):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args], cwd=ROOT, capture_output=True,
                          text=True, timeout=timeout)


def test_more_than_one_gpu_is_refused_with_a_message():
    r = run_bench("--gpus", "2")
    assert r.returncode != 0
    assert "single-GPU" in r.stderr and r.stdout.strip() == ""


def test_measured_traffic_belongs_to_every_source_of_the_gemms(tmp_path):
    # the measured traffic is reported only for the kernels it was measured on: the guard covers the file that holds the
    # kernel, the one that launches it, and all of this library's headers that they include
    import bench
    holders = [n for n in os.listdir(CSRC) if "panel_gemm_kernel" in open(os.path.join(CSRC, n)).read()
               or "launch_gate_up(a" in open(os.path.join(CSRC, n)).read()]
    assert {"ffn.hip", "ffn_gemm.hip"} <= set(holders)
    sources, todo = set(), holders
    while todo:
        name = todo.pop()
        sources.add(name)
        included = re.findall(r'#include "([^"]+)"', open(os.path.join(CSRC, name)).read())
        todo += [n for n in included if n not in sources and os.path.exists(os.path.join(CSRC, n))]
    assert sources <= set(bench.TRAFFIC_SOURCES)
    now = bench._traffic_sources_sha256()
    for name in bench.TRAFFIC_SOURCES:
        copy = tmp_path / name.replace(".", "_")
        shutil.copytree(CSRC, copy)
        assert bench._traffic_sources_sha256(str(copy)) == now
        with open(copy / name, "a") as fh:
            fh.write("\n")
        assert bench._traffic_sources_sha256(str(copy)) != now, name


def test_garbage_of_the_setup_is_not_collected_in_the_timed_steps(monkeypatch):
    # a full collection takes 40 ms with torch loaded; made due by the set-up, it fell into the timed steps of some runs
    import gc
    import types
    import torch
    import bench
    from paper_2604_19654_amd import binding, runner
    due = []

    class Clocked(Exception):
        pass

    def step(p, mark, early_static):
        p.layer.timeline = dict(p.layer.timeline, start=None)
        due.append(gc.get_count()[1:])
        if len(due) == 3:      # two warm-up steps, the first timed one
            raise Clocked

    def prepare(*a, **k):
        return types.SimpleNamespace(wl=None, layer=types.SimpleNamespace(timeline={}))
    monkeypatch.setattr(runner, "prepare", prepare)
    monkeypatch.setattr(runner, "step", step)
    monkeypatch.setattr(binding, "HipEvent", lambda: [[] for _ in range(2000)])     # garbage: more than a young collection's worth
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    with pytest.raises(Clocked):
        bench.time_workload("C1", 20, 2)
    assert due[2] == (0, 0), "collections were due when the clock started"


@pytest.mark.gpu
def test_one_json_line_with_the_agreed_keys():
    r = run_bench("--workload", "C1", "--steps", "3", "--warmup", "1", "--cpu-tokens", "256")
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [ln for ln in r.stdout.splitlines() if ln.strip()]
    assert len(lines) == 1
    d = json.loads(lines[0])
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert key in d, key
    assert d["n_gpus"] == 1 and d["steps"] == 3 and d["warmup"] == 1 and d["higher_is_better"] is True
    assert d["unit"] == "TFLOP/s" and d["dtype"] == "bf16" and d["data"] == "synthetic" and d["vs_baseline"] is None
    assert d["config"]["workload"].startswith("C1") and "model" not in d["config"]
    roof = d["roofline"]
    assert roof["bound"] == "mfma" and roof["unit"] == "TFLOP/s" and roof["peak"] == 2500.0
    assert abs(roof["frac"] - roof["achieved"] / roof["peak"]) < 1e-12
    cpu = d["cpu_baseline"]
    assert cpu["kind"] == "oracle" and cpu["cores"] >= 1 and cpu["value"] > 0 and cpu["integer_outputs_match"] is True
    assert d["value"] > 0 and d["ms_per_step"] > 0
    assert cpu["parity"] is True and cpu["rows_above_row_bar"] == 0 and cpu["worst_element_over_storage_format_bound"] <= 1.0
    assert cpu["host_cpus"] >= cpu["cores"] >= 1
    # one roofline object per kernel of the step, each recomputable from its own fields
    assert set(d["rooflines"]) == {"down", "combine", "permute_with_gather", "row_gather_alone", "route"}
    for key, r in list(d["rooflines"].items()) + [("gate_up", roof)]:
        assert r["bound"] in ("mfma", "hbm", "alu") and abs(r["frac"] - r["achieved"] / r["peak"]) < 1e-9, key
        assert r["avg_launch_ms"] > 0
    assert roof["per_launch"][0]["nonempty_groups"] == d["config"]["nonempty_groups"] == 8
    assert abs(roof["flops_per_launch"] / (roof["avg_launch_ms"] * 1e-3) / 1e12 - roof["achieved"]) < 1e-6 * roof["achieved"]
    # the other four workloads are timed in the default run as well
    assert set(d["other_workloads"]) == {"C2", "C3", "C4", "C5"}
    c3 = d["other_workloads"]["C3"]
    assert c3["gate_up"]["frac"] > 0 and c3["down"]["frac"] > 0 and c3["R"] > 8192
    assert d["ffn_training_step"]["ms"]["backward"] > 0
