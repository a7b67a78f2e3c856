"""The benchmark's output is one JSON line that a reader of the last few thousand characters still gets whole."""
import json

import bench

CONTRACT = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
            "dtype", "data", "config")


def measured(name):
    """A workload's result with every field the run fills in, at full float length."""
    x = 1234567.0 / 7.0
    kernels = {k: {"avg_us": x, "launches": 52, "GBps": x, "TFLOPps": x} for k in bench.KIND_BOUND}
    roof = {"bound": "mfma", "kernel": "ffn_gate_up_kernel (weight streaming)", "achieved": x, "peak": 2500.0, "unit": "TFLOP/s",
            "frac": x, "traffic": x, "traffic_source": "profiles/ffn_kernels_mixtral_decode_T64_pmc_traffic.md", "avg_launch_us": x,
            "alg_flops_per_launch": x, "launches": 384, "share_of_step_time": x, "measured_peak": x, "frac_of_measured_peak": x}
    base = {"value": x, "unit": "tokens/s", "cores": 16, "sample": "s" * 140}
    return {"name": name, "baseline_config": 2, "note": "n" * 120, "value": x, "unit": "tokens/s", "steps": 20, "warmup": 5,
            "ms_per_step": x, "dtype": "bf16",
            "config": {"workload": "w" * 170, "tokens_per_step": 64, "layers": 32, "beta": 16.0, "horizon": "adaptive",
                       "drift_tokens": 0},
            "us_per_layer": x, "ms_per_step_p10_p50_p90": [x] * 3, "stall_frac": x, "hit_rate": x,
            "beta_changed_token_frac": x, "link_bound_bytes_per_layer": x, "expert_bytes": 352321536,
            "cache": {f"statistic_{i}": x for i in range(24)}, "kernels": kernels, "token_dist": x, "roofline": roof,
            "cpu_baseline": dict(base, kind="oracle", single_thread=base)}


def test_line_is_short_and_whole():
    peaks = {"hbm_read_GBps": 6543.21, "mfma_16bit_TFLOPps": 2212.3, "pcie_h2d_GBps": 57.1, "published": {"hbm_GBps": 8000.0},
             "how": "h" * 200}
    results = [measured(n) for n in bench.DEFAULT_SET]
    line = json.dumps(bench.line_of(results, peaks, False, True))
    assert len(line) < 6000 and "\n" not in line
    got = json.loads(line)
    assert all(k in got for k in CONTRACT)
    assert got["value"] == results[0]["value"] and got["ms_per_step"] == results[0]["ms_per_step"]
    assert [w["name"] for w in got["workloads"]] == bench.DEFAULT_SET
    assert abs(got["workloads"][3]["value"] - results[3]["value"]) <= 1e-4 * results[3]["value"]
    full = bench.line_of(results, peaks, True, True)
    assert full["workloads"] == results and full["kernels"] == results[0]["kernels"]
    one = bench.line_of(results[:1], peaks, False, False)
    assert "workloads" not in one and one["roofline"]["kernel"] == results[0]["roofline"]["kernel"]
