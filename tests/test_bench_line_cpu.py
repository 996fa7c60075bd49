"""The bench's one line: the contract's keys, whole in the few kilobytes that a log's tail keeps,
however many kernels, arms and workloads were measured."""
import json

import bench


def _record(extra=True):
    kernels = {f"prefix.kernel_number_{i}": {"launches": 12, "avg_ms": 1.23456789012345, "ms_per_step": 4.93827156049380}
               for i in range(40)}
    roof = {"kernel": "prefix.gemm_gate_up (fused SwiGLU)", "bound": "mfma", "achieved": 1296.5687754179742,
            "peak": 2500.0, "unit": "TFLOP/s", "frac": 0.5186275101671897, "traffic": 29040223210.3586,
            "algorithmic_per_launch": 18554258718720.0, "algorithmic_per_unit": "2 * 2F * d flop per prefix token",
            "algorithmic_bytes_per_launch": 2713714688, "frac_of_measured_peak": 0.730}
    rec = {"metric": "prefix prefill tokens/s + suffix logprob tokens/s; % bf16 MFMA peak", "value": 515220.1257861635,
           "unit": "tokens/s", "n_gpus": 1, "steps": 20, "warmup": 3, "ms_per_step": 65.58750152587890,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
           "config": {"workload": "qwen32b_b2_p16384_s512", "layers": 2, "d_model": 5120, "parallelism": "single GPU"},
           "prefix_ms": 61.167503356933594, "prefix_mfma_frac": 0.4898346123024439, "roofline": roof,
           "logsoftmax_roofline": roof, "step_ms": {"median": 65.59520721435547}, "kernels": kernels}
    if extra:
        rec["workloads"] = {f"workload_{i}": _record(False) for i in range(2)}
        rec["transposed_weights_variant"] = {"value": 515342.7047555221, "unit": "tokens/s", "kernels": kernels}
        rec["colocation"] = {"metric": "m", "value": 297813.71835427784, "arms": [dict(roof) for _ in range(9)],
                             "config": {"workload": "coloc"}, "decode_kernels": kernels, "prefix_alone_ms": 57.583}
    return rec


def test_the_line_is_short_and_keeps_the_contract():
    rec = _record()
    line = json.dumps(bench.brief(rec))
    assert len(line) < 5000
    got = json.loads(line)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config", "roofline", "workloads", "colocation"):
        assert key in got
    assert abs(got["value"] / rec["value"] - 1) < 1e-5 and got["config"] == rec["config"]
    assert got["workloads"]["workload_1"]["prefix_ms"] and got["colocation"]["prefix_alone_ms"]
    assert got["roofline"]["frac"] == 0.518628
