"""CPU checks of the benchmark's contract: it measures one GPU only and says
so when asked for more (before touching a device), and the memory-counter
traffic it reports still belongs to the roofline kernel's current source."""
import os
import subprocess
import sys

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(args, env=None):
    e = dict(os.environ)
    e.update(env or {})
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args], cwd=ROOT,
                          capture_output=True, text=True, env=e, timeout=120)


def test_more_than_one_gpu_is_refused():
    r = _run(["--gpus", "2"])
    assert r.returncode == 2
    assert "one GPU" in r.stderr
    assert r.stdout == ""


def test_a_distributed_launch_is_refused():
    r = _run([], env={"WORLD_SIZE": "2"})
    assert r.returncode == 2 and "one GPU" in r.stderr


def test_counter_traffic_is_reported_only_for_the_current_kernel():
    # counters are reported only for the kernel they were taken on, and only
    # while its source region hashes as it did then; otherwise None
    import hashlib
    import json

    with open(os.path.join(ROOT, "profiles", "roofline_traffic.json")) as f:
        data = json.load(f)
    with open(os.path.join(ROOT, data["source_file"])) as f:
        text = f.read()
    for workload, e in data["workloads"].items():
        begin, end = e["source_region"]
        current = begin in text and end in text and hashlib.sha256(
            text[text.index(begin):text.index(end)].encode()).hexdigest() == e["source_sha256"]
        for kernel in e["kernels"]:
            t = bench.counter_traffic(workload, kernel)
            assert (t is not None and t > 0) if current else t is None, (workload, kernel)
        assert bench.counter_traffic(workload, "k_no_such_kernel") is None
    assert bench.counter_traffic("no_such_workload", "k_csr<2, 16, double>") is None


def test_the_printed_line_is_short_and_keeps_the_contract(tmp_path, capsys):
    """Whatever the legs hold, the printed line is one JSON object that the last
    2,000 characters of a log hold whole; the full record is in the file."""
    import json

    long = {"value": 123.456789012345, "note": "x" * 300, "top_kernels": [{"kernel": "k" * 40}] * 8}
    out = {"metric": bench.METRIC, "value": 222.123456789012, "unit": "solves/s", "n_gpus": 1,
           "steps": 20, "warmup": 5, "ms_per_step": 4.44444444444444, "higher_is_better": True,
           "scaling": "weak", "vs_baseline": None, "dtype": "f64", "data": "synthetic",
           "config": dict({"workload": "w" * 340}, **{f"figure_number_{k}": 1.0 / 3 for k in range(9)}),
           "roofline": dict({k: 1.0 / 3 for k in bench.LINE_ROOFLINE}, kernel="k_csr<2, 8, double>",
                            top_kernels=[long] * 8),
           "cpu_baseline": dict(long, unit="solves/s", cores=1, kind="oracle", host_cpu="AMD EPYC"),
           "variants": {"c5_plate": {"mixed_learned": long, "mixed_zero_guess": long, "other": long},
                        "c3_128cube": {"fp64": dict(solves_per_s=133.25), "mixed": long}, "c4_uq_batched": long,
                        "c2_64cube": {"mixed_learned": long}}}
    path = tmp_path / "detail.json"
    bench.report(out, str(path))
    text = capsys.readouterr().out
    assert text.count("\n") == 1 and len(text) <= bench.LINE_CHARS
    line = json.loads(text)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
              "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config"):
        assert k in line, k
    assert abs(line["value"] - out["value"]) <= 1e-5 * out["value"]
    assert line["variants"]["c4_uq_batched"] == 123.457 and len(line["variants"]) == 6
    assert line["variants"]["c3_128cube.fp64"] == 133.25
    with open(path) as f:
        assert json.load(f) == out
    bench.report({k: v for k, v in out.items() if k not in ("variants", "roofline", "cpu_baseline")},
                 "")
    assert "detail" not in json.loads(capsys.readouterr().out)
