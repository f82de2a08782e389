"""bench.py's command line, on the CPU: the options parse, and a request for
more than one GPU, or for a workload that is not a whole decoder layer, ends
with a message before any GPU work."""
import importlib.util
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench(*args):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), *args],
                          stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True, timeout=120)


def test_help_lists_the_options():
    p = _bench("--help")
    assert p.returncode == 0
    for opt in ("--gpus", "--steps", "--warmup", "--ratios", "--no-cpu-baseline",
                "--no-fused-attention", "--no-decode", "--copy-probe-mib", "--no-policies",
                "--no-attention-chain", "--no-mlp-chain", "--no-pv", "--no-paper-kernels",
                "--no-layer-forward", "--no-decode-batched", "--workload", "--records"):
        assert opt in p.stdout


def test_more_than_one_gpu_is_refused():
    p = _bench("--gpus", "2")
    assert p.returncode == 2
    assert "one GPU" in p.stderr


def test_parity_workloads_are_refused():
    # the step is a whole decoder layer; the single-product workloads are
    # parity-test cases, refused before any GPU work
    for wk in ("mlp_1b", "linear_f32", "attn_4k", "no_such_workload"):
        p = _bench("--workload", wk)
        assert p.returncode != 0
        assert wk in p.stderr


def test_line_is_short_and_keeps_the_headline():
    """The printed line keeps every contract key and each record's rooflines
    and entries at the headline ratio, without the tables and descriptions."""
    spec = importlib.util.spec_from_file_location("_bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    row = {f"key_{i}": 123.456 for i in range(14)}
    times = dict.fromkeys(("ms_per_step", "tflops", "gemm_tflops", "speedup_vs_r1"), 1.5)
    ratios = ("0.25", "0.5", "0.75", "1.0")
    roof = {"bound": "hbm", "kernel": "k" * 60, "achieved": 1.0, "peak": 2.0, "unit": "GB/s", "frac": 0.5}
    out = {"metric": "m", "value": 1.0, "config": {"r": 0.5}, "sweep": {r: {**row, **times} for r in ratios}}
    for name in ("fused_attention", "decode", "pv_chain", "mlp_chain"):
        out[name] = {"op": "x" * 400, "kernels": ["k"] * 9, "per_ratio": dict.fromkeys(ratios, row),
                     "speedup_vs_r1": 1.5, "roofline": roof}
    out["norm_chain"] = {"op": "x" * 300, "per_input_ratio": {f"{i}@{r}": row for i in "ab" for r in ratios}}
    out["decode_batched"] = {"op": "x" * 300, "per_batch_ratio": {f"B{b}@{r}": row for b in (4, 16, 32) for r in ratios}}
    out["paper_kernels"] = {"op": "x" * 500, "per_length": dict.fromkeys(("1024", "2048", "4096"), row)}
    out["layer_forward"] = {"op": "x" * 300, "per_ratio": {"rmm_ms@0.5": 2.0, "rmm_ms@1.0": 3.0, "dense_ms": 5.0}}
    out["component_ratios"] = {"op": "x" * 200, "policies": {"p": {**row, **times}}}
    line = bench.summary(out)
    assert len(json.dumps(line)) < 9000 < len(json.dumps(out))
    assert line["value"] == 1.0 and line["config"] == {"r": 0.5}
    assert list(line["sweep"]) == list(ratios) and set(line["sweep"]["1.0"]) == set(times)
    assert line["decode"] == {"per_ratio": {"0.5": row}, "speedup_vs_r1": 1.5, "roofline": roof}
    assert list(line["norm_chain"]["per_input_ratio"]) == ["a@0.5", "b@0.5"]
    assert list(line["decode_batched"]["per_batch_ratio"]) == ["B4@0.5", "B16@0.5", "B32@0.5"]
    assert list(line["paper_kernels"]["per_length"]) == ["1024", "2048", "4096"]
    assert line["component_ratios"] == {"p": times}
    assert line["layer_forward"] == {"per_ratio": {"rmm_ms@0.5": 2.0}}
    assert out["decode"]["op"]                                # the record itself is left whole
