"""Host-side pieces of bench.py (no GPU): the counter-summary lookup, the
multi-GPU refusal and the CPU model of the baseline."""
import hashlib
import os
import subprocess
import sys

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _fake_tree(tmp_path, kernel_src, sha, lines):
    (tmp_path / "profiles").mkdir()
    (tmp_path / "paper_1902_00088_amd" / "csrc").mkdir(parents=True)
    (tmp_path / "paper_1902_00088_amd" / "csrc" / "kernels.hip").write_bytes(kernel_src)
    text = "# counters\n\ntraffic_sha256: " + sha + "\n" + "\n".join(lines) + "\n"
    (tmp_path / "profiles" / "stage_traffic_counters.md").write_text(text)


def test_counter_traffic_reads_the_line_of_the_tiling_while_the_source_matches(tmp_path, monkeypatch):
    src = b"// kernel source\n"
    sha = hashlib.sha256(src).hexdigest()
    _fake_tree(tmp_path, src, sha, ["traffic_bytes_per_launch c2 nsub 4: 2047807",
                                    "traffic_bytes_per_launch c2 nsub 1 t512: 2094173"])
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.counter_traffic("c2 nsub 4") == 2047807.0
    assert bench.counter_traffic("c2 nsub 1" + bench.tkey({"stage_threads": 512})) == 2094173.0
    assert bench.counter_traffic("c2 nsub 2") is None          # not measured
    assert bench.tkey({"stage_threads": 256}) == "" and bench.tkey({}) == ""


def test_traffic_key_names_the_kernel_the_run_used():
    stage = {"stage_tiles": 4, "stage_threads": 256}
    assert bench.traffic_key("c2", stage, "stage") == "c2 nsub 4"
    tile = {"rk4_tile": {"tiles": 2, "analysis_folded": [1, 1024], "refine_folded": [1, 1, 512],
                         "mothers_folded": [1, 256]}}
    assert bench.traffic_key("c2", tile, "rk4_tile") == "c2 rk4_tile nsub 1 t256 analysis refine mothers"
    tile["rk4_tile"]["mothers_folded"] = [0, 256]
    assert bench.traffic_key("c2", tile, "rk4_tile") == "c2 rk4_tile nsub 1 t512 analysis refine"
    tile["rk4_tile"]["refine_folded"] = [0, 1, 512]
    assert bench.traffic_key("c2", tile, "rk4_tile") == "c2 rk4_tile nsub 1 t1024 analysis"
    tile["rk4_tile"]["analysis_folded"] = [-1, 256]
    assert bench.traffic_key("c2", tile, "rk4_tile") == "c2 rk4_tile nsub 2"
    assert bench.traffic_key("c2", stage, "mr") is None and bench.counter_traffic(None) is None


def test_counter_traffic_is_void_once_the_kernel_source_changes(tmp_path, monkeypatch):
    src = b"// kernel source\n"
    _fake_tree(tmp_path, src, hashlib.sha256(b"// older source\n").hexdigest(),
               ["traffic_bytes_per_launch c2 nsub 4: 2047807"])
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.counter_traffic("c2 nsub 4") is None


def test_committed_counter_summary_parses():
    """The committed summary has a hash line and at least one figure per workload."""
    text = open(os.path.join(ROOT, "profiles", "stage_traffic_counters.md")).read()
    assert any(l.startswith("traffic_sha256: ") for l in text.splitlines())
    for w in ("c2", "c4"):
        vals = [float(l.split(":", 1)[1]) for l in text.splitlines()
                if l.startswith(f"traffic_bytes_per_launch {w} nsub ")]
        assert vals and all(v > 0 for v in vals)


def test_bench_refuses_more_than_one_gpu():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr


def test_cpu_model_names_the_host_processor():
    name = bench.cpu_model()
    assert name is None or (isinstance(name, str) and name.strip())
    if name and os.path.exists("/proc/cpuinfo"):
        want = next((ln.split(":", 1)[1].strip() for ln in open("/proc/cpuinfo") if ln.startswith("model name")), None)
        if want:
            assert name.startswith(want)


def test_traffic_key_tells_splits_of_blocks_apart():
    """Halves and thirds of blocks are other kernels than whole ones of as many threads."""
    form = {"stage_tiles": 1, "stage_threads": 512, "stage_parts": 3}
    assert bench.traffic_key("c3", form, "stage") == "c3 nsub 1 t512 p3"
    assert bench.traffic_key("c3", dict(form, stage_parts=1), "stage") == "c3 nsub 1 t512"


def test_counter_traffic_is_void_once_any_kernel_source_changes(tmp_path, monkeypatch):
    """Workgroup sizes and argument layouts stand in headers: the summary's hash covers them."""
    src = b"// kernel source\n"
    names = ("column3.hip", "plane2.hip", "device.hpp", "internal.hpp")
    sha = hashlib.sha256(src + b"".join(n.encode() for n in names)).hexdigest()
    _fake_tree(tmp_path, src, sha, ["traffic_bytes_per_launch c2 nsub 4: 2047807"])
    csrc = tmp_path / "paper_1902_00088_amd" / "csrc"
    for n in names:
        (csrc / n).write_bytes(n.encode())
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.counter_traffic("c2 nsub 4") == 2047807.0
    for n in names:
        (csrc / n).write_bytes(b"changed")
        assert bench.counter_traffic("c2 nsub 4") is None, n
        (csrc / n).write_bytes(n.encode())


def test_printed_line_is_short_and_keeps_the_headline():
    """The line holds every headline field as measured and a summary of the rest, in less than
    the 4 KiB that a reader of a run's tail surely has; the whole record takes many times that."""
    import argparse
    import json
    kernels = {k: {"launches": 80, "ms": 0.8416951234567, "bytes": 1605795840.0}
               for k in ("stage", "ghost", "rhs_plain", "rk4_tile", "mr", "refine", "coarsen", "topology", "read")}
    form = {"value": 3543684.2133620796, "ms_per_step": 0.01806030000039982, "block_updates": 1280, "blocks_initial": 16,
            "blocks_final": 16, "sweep_block_updates_per_s": 5.04e6, "kernels": kernels, "stage_tiles": 1,
            "stage_threads": 384, "stage_parts": 1, "sweep_launch": "rk4_tile",
            "host_us_per_step": {f"phase{i}": 0.1234567890123 for i in range(12)},
            "tune_ms": {f"key{i}": 0.1234567890123 for i in range(60)}, "rk4_tile": {"tiles": 1}}
    forms = {n: dict(form) for n in ("fp64_plain", "fp64_fused", "mixed_fused")}
    acc = {"steps": 20, "topology": "FP64 run's flags replayed", "same_forest": True, "max_rel_inf": 3.04376123456789e-08,
           "rel_inf_per_field": {"phi": 1e-9}, "rel_l2_per_field": {"phi": 1e-9}, "within_1e-5": True}
    args = argparse.Namespace(steps=20, warmup=5)
    out = bench.headline(args, forms, acc)
    for w in ("c4", "c3"):
        out[w] = {"workload": "w" * 140, "forms": forms, "mixed_accuracy": acc,
                  "speedup_mixed_fused_vs_fp64_plain": bench.speedup_entry(forms, acc),
                  "speedup_mixed_fused_vs_fp64_fused": bench.speedup_entry(forms, acc, base="fp64_fused"),
                  "roofline_stage_mixed": dict(out["roofline"])}
    study = {"test_accuracy": 0.5794371234, "block_updates_saved": 0.20192645825631406, "within_bound": False,
             "degenerate": False, "guards": {"0.0": {f"k{i}": 0.123456789 for i in range(40)}}}
    out["predictor"] = {"C5_mixing_layer": study, "swirl_moving_fronts": study}
    out["cpu_baseline"] = {"value": 13383.8, "unit": "block-updates/s", "cores": 16, "kind": "oracle", "sample": "s" * 110,
                           "cpu_model": "m" * 60, "host_threads_available": 16,
                           "single_thread": {"value": 1116.98, "cores": 1, "sample": "s" * 90}}
    line = json.dumps(bench.summary(out))
    assert len(line) < 4096 < len(json.dumps(out)) / 3
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config"):
        assert got[k] == out[k], k
    assert set(got) == set(out) and got["roofline"]["kernel"] == out["roofline"]["kernel"]
    assert got["c3"]["forms"]["mixed_fused"]["ms_per_step"] == 0.0180603
    assert got["predictor"]["C5_mixing_layer"]["block_updates_saved"] == 0.201926
    assert bench.summary({}) == {} and bench.summary({"mixed_accuracy": None}) == {"mixed_accuracy": None}
