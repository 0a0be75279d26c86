"""bench.py's command line and the JSON line it prints: the keys and types the driver reads.
The GPU case runs a short bench (few steps) on the metric's workload."""
import glob
import json
import os
import re
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BENCH = os.path.join(ROOT, "bench.py")


def test_more_than_one_gpu_is_refused_with_a_message():
    r = subprocess.run([sys.executable, BENCH, "--gpus", "2"], capture_output=True, text=True, timeout=120)
    assert r.returncode != 0
    assert "one gpu" in r.stderr.lower() and r.stdout.strip() == ""


def test_counter_readings_that_the_memory_could_not_carry_are_not_reported():
    sys.path.insert(0, ROOT)
    import bench
    assert bench.plausible_traffic(None, 0.03) == (None, None)
    got, source = bench.plausible_traffic(150e6, 0.03)          # 5 TB/s
    assert got == 150e6 and source.startswith("offline")
    got, source = bench.plausible_traffic(239e6, 0.024)         # 10 TB/s
    assert got is None and source.startswith("stale")
    assert bench.plausible_traffic(239e6, 0.0)[0] is None


def test_profiles_name_kernels_of_the_library():
    """Every kernel that a summary under profiles/ names is one the built library holds: figures of a kernel
    that another has replaced are figures of an older build."""
    lib = os.path.join(ROOT, "paper_2411_05289_amd", "libmdsd.so")
    if not os.path.exists(lib) or shutil.which("nm") is None:
        pytest.skip("needs the built library and nm")
    names = subprocess.run(["nm", "-C", lib], capture_output=True, text=True, check=True).stdout
    have = {re.sub(r"^void ", "", l.split(" ", 2)[2]).split("(")[0]
            for l in names.splitlines() if "mdsd" in l and re.match(r"[0-9a-f]+ \w ", l)}
    seen = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "profiles", "*.txt"))):
        for name in re.findall(r"mdsd\w*::\w+(?:<[^>]*>)?", open(path).read()):
            if name != "mdsd::Params":
                assert name in have, (os.path.basename(path), name)
                seen += 1
    assert seen > 50


@pytest.mark.gpu
@pytest.mark.parametrize("config", ["2", "toy"])
def test_bytes_moved_stay_below_the_memory_peak(config):
    r = subprocess.run([sys.executable, BENCH, "--config", config, "--steps", "20", "--warmup", "5", "--no-cpu-baseline",
                        "--no-path-only"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    roof = json.loads(r.stdout)["roofline"]
    assert roof["traffic_source"].startswith("offline") and 0 < roof["frac_of_bytes_moved"] < 1


@pytest.mark.gpu
def test_json_line_of_a_short_run():
    r = subprocess.run([sys.executable, BENCH, "--steps", "20", "--warmup", "5"],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [l for l in r.stdout.splitlines() if l.strip()]
    assert len(lines) == 1
    d = json.loads(lines[0])
    assert d["unit"] == "nodes/s" and d["n_gpus"] == 1 and d["steps"] == 20 and d["warmup"] == 5
    assert d["higher_is_better"] is True and d["vs_baseline"] is None and d["data"] == "synthetic"
    assert d["config"]["workload"].startswith("V32000_B64") and "model" not in d["config"]
    assert d["value"] > 0 and d["ms_per_step"] > 0
    assert abs(d["value"] - 64 * 31 / (d["ms_per_step"] * 1e-3)) < 1e-6 * d["value"]
    roof = d["roofline"]
    assert roof["bound"] == "hbm" and roof["unit"] == "GB/s" and roof["peak"] == 8000.0
    assert abs(roof["frac"] - roof["achieved"] / roof["peak"]) < 1e-12
    assert roof["algorithmic_bytes_per_launch"] == 64 * (31 + 15) * 32000 * 2
    assert abs(roof["achieved"] - roof["algorithmic_bytes_per_launch"] / (roof["kernel_ms"] * 1e-3) / 1e9) < 1e-6 * roof["achieved"]
    assert 0.2 < roof["frac"] < 1.0          # a kernel faster than the memory could feed it would be a bug
    cpu = d["cpu_baseline"]
    assert cpu["kind"] == "oracle" and cpu["unit"] == "nodes/s" and cpu["value"] > 0 and cpu["cores"] >= 1
    assert d["path_only"]["trees_per_s"] > 0


@pytest.mark.gpu
@pytest.mark.parametrize("args,kernel", [([], "spechub_step"), (["--walk-in-verify"], "spechub_verify")])
def test_the_roofline_is_of_what_is_timed(args, kernel):
    """A step in one call beside the draft and the verify call one after the other, each under its own name."""
    r = subprocess.run([sys.executable, BENCH, "--steps", "50", "--warmup", "5", "--no-cpu-baseline"] + args,
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    d = json.loads(r.stdout)
    assert d["roofline"]["kernel"] == kernel and d["roofline"]["kernel_ms"] <= 1.05 * d["ms_per_step"]
    two = d["draft_then_verify"]
    assert set(two["kernels"]) == {"spechub_draft", "spechub_verify"}
    assert abs(two["nodes_per_s"] - 64 * 31 / (two["ms_per_step"] * 1e-3)) < 1e-6 * two["nodes_per_s"]
    assert sum(k["kernel_ms"] for k in two["kernels"].values()) <= 1.05 * two["ms_per_step"]
    if args:
        assert two["ms_per_step"] == d["ms_per_step"]
