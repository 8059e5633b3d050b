"""The benchmark's line holds its keys and stays short, however large the tables are (no compute: this runs without a GPU)."""
import json

import bench


def record():
    row = {"K": 14336, "N": 28672, "M": 256, "us": 123.45, "tflops": 1234.56, "gbs": 1234.5, "frac_mfma": 0.1234, "frac_hbm": 0.1234, "frac_roofline": 0.1234}
    steps = [{"B": b, "context": 512, "ms_per_step": 0.621, "tokens_per_s": 103141.4} for b in (1, 8, 64)]
    job = {"prompts": 64, "seconds_each_run": [0.0933] * 3, "generated_tokens_per_s": 87714.1}
    return {
        "metric": "m" * 80, "value": 1.0, "unit": "TFLOP/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 1.0, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic", "config": {"workload": "w" * 240, "launches_per_step": 36, "flop_per_step": 2e11},
        "roofline": {"kernel": "k" * 80, "per_shape": [{"K": 14336, "N": 28672, "min_frac_hbm_M_le_8": 0.1234, "min_frac_mfma_M_ge_128": 0.1234,
                                                       "min_frac_mfma_M_ge_128_fixed_tile": 0.1234}] * 4},
        "fingerprint": "f" * 320, "measured_peaks": {"copy_1GiB_gbs": 5170.1, "read_1GiB_gbs": 4000.1, "same_bytes": [row] * 4},
        "cpu_baseline": {"value": 0.1, "sample": "s" * 120, "other_legs": [row] * 40}, "bit_identical": {"rate": 1.0, "comparisons": 180, "what": "b" * 100},
        "sweep_cold": [row] * 36, "sweep_warm": [row] * 36, "sweep_cold_fixed_tile": [row] * 36, "attention": [row] * 16, "library_gemm": [row] * 36,
        "qgemm_w4a8": [row] * 20, "token_selection": [row] * 16,
        "decode": {"decoder_layer": [{"B": 1, "layer_tokens_per_s": 9622.0}] * 3, "model_8_layer_step": steps, "model_8_layer_step_w4a8": steps, "job_64_prompts": job},
    }


def test_the_line_is_short_and_whole():
    r = record()
    line, tables = bench.split_record(r)
    assert len(json.dumps(line)) <= bench.LINE_BYTES < len(json.dumps(r))
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "config",
              "roofline", "fingerprint", "bit_identical"):
        assert line[k] == r[k]
    assert line["cpu_baseline"]["value"] == 0.1 and r["cpu_baseline"]["other_legs"] == tables["cpu_baseline_other_legs"]
    assert line["decode_tokens_per_s"] == {"model_8_layer_step": {"B1": 103141.4, "B8": 103141.4, "B64": 103141.4},
                                           "model_8_layer_step_w4a8": {"B1": 103141.4, "B8": 103141.4, "B64": 103141.4}, "job_64_prompts": 87714.1}
    for k in r:
        assert k in line or k in tables
    assert "same_bytes" in tables["measured_peaks"]


def test_a_short_run_has_a_line_too():
    r = {k: v for k, v in record().items() if k not in ("measured_peaks", "cpu_baseline", "bit_identical", "decode")}
    line, _ = bench.split_record(r)
    assert line["value"] == 1.0 and line["decode_tokens_per_s"] == {}
