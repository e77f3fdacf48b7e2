"""bench.py's printed line: the contract's fields, and short enough that a reader who keeps the end of the output has it all."""
import json

import bench


def _record(name):
    series = {"per_step": [0.123] * 20}
    roof = {"bound": "mfma", "achieved": 847.25, "peak": 2500.0, "unit": "TFLOP/s", "frac": 0.3389, "kernel": "attn_mfma_kernel",
            "traffic": None, "avg_launch_ms": 12.5, "measured": "x" * 120, "sclk_MHz_during_timed_steps": {"median": 1900.0}}
    return {"metric": "tokens/s of paged multi-LoRA layer step", "value": 2.1e6, "unit": "tokens/s", "n_gpus": 1, "steps": 20,
            "warmup": 5, "ms_per_step": 17.8, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
            "dtype": "bf16", "data": "synthetic",
            "config": {"workload": name, "swap": "y" * 200, "trace": {"mode": "bursty", "replaced_slots_per_step": [4] * 200,
                                                                     "distinct_adapters_per_step": [200] * 200}},
            "roofline": roof, "step_pace_ms": [17.8] * 200, "swap_traffic": series, "serialised": series,
            "kernels": {k: dict(roof) for k in ("swap", "lora_qkv", "kv_append", "attention", "lora_o")},
            "cpu_baseline": {"value": 100.0, "note": "z" * 100}}


def test_the_printed_line_keeps_the_contract_and_stays_short():
    rec = _record("34b_gqa")
    rec["sub_records"] = {n: _record(n) for n in bench.WORKLOADS[1:]}
    rec["host_logic"] = {"full": {"x": "y" * 400}, "lru": {"x": "y" * 400}}
    line = json.dumps(bench.summary(rec))
    assert len(json.dumps(rec)) > 20000 and len(line) < 4000 and "\n" not in line
    out = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config", "roofline"):
        assert out[k] == rec[k] or k == "config", k
    assert out["config"]["workload"] == "34b_gqa" and out["config"]["trace"] == {"mode": "bursty"}
    assert set(out["sub_records"]) == set(bench.WORKLOADS[1:]) and out["sub_records"]["tiny"]["ms_per_step"] == 17.8
