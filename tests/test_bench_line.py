"""The line bench.py prints holds the headline and stays short whatever was measured beside it: a record of the
output's end must hold all of it."""
import json

import bench


def _config(n):
    kernels = {f"kernel_number_{i}": {f"field_{j}": 123456.789 for j in range(16)} for i in range(n)}
    roof = {k: 1234.5678 for k in bench.ROOFLINE_FIELDS} | {"kernel": "gated_attention_bwd_tokens", "cache": "c" * 300}
    return {"workload": "w" * 120, "value": 123456789.123456789, "unit": "selected tokens/s", "ms_per_step": 0.0305404999,
            "ms_per_step_min": 0.0293996, "launch": "l" * 400, "kernels": kernels, "roofline": roof,
            "single_stream": {"ms_per_step": 0.04, "value": 1e8, "cache": "c" * 100}}


def test_the_printed_line_is_short_and_whole():
    head = _config(3)
    configs = {name: _config(8) for name in ("det", "tiny", "vit_s", "vit_b_train", "hierarchy")}
    configs["hierarchy"]["forward"] = _config(8)
    result = {"metric": "selected tokens/sec (SPA fwd) at 1 GPU", "value": head["value"], "unit": head["unit"], "n_gpus": 1,
              "steps": 200, "warmup": 50, "ms_per_step": head["ms_per_step"], "higher_is_better": True, "scaling": "weak",
              "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
              "config": {"workload": "w" * 120, "selected_tokens": 8491, "launch": "l" * 400, "timing": "t" * 100},
              "ms_per_step_min": 0.029, "ms_per_step_until_last_event": 0.03, "single_stream": head["single_stream"],
              "roofline": head["roofline"], "ceilings": {"copy_GBs": 5506.1, "copy": "c" * 100}, "kernels": head["kernels"],
              "configs": configs, "extras": {"padded_baseline": {"packed_attention_us": 30.17, "padded_dense_us": 55.51,
                                                                    "padded_skipping_masked_keys_us": 36.52, "text": "t" * 400},
                                                "other": configs},
              "cpu_baseline": {"value": 22052.18, "unit": "selected tokens/s", "cores": 16, "kind": "oracle", "sample": "s" * 80}}
    line = json.dumps(bench.summary(result))
    assert len(line) < 2000 and "\n" not in line
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data"):
        assert got[k] == result[k], k
    assert got["config"]["workload"] == result["config"]["workload"] and got["roofline"]["kernel"] == head["roofline"]["kernel"]
    assert got["cpu_baseline"]["value"] == result["cpu_baseline"]["value"]
    assert set(got["configs"]) == {*configs, "hierarchy_forward"}
    assert all(abs(c["value"] - head["value"]) < 0.1 and c["us"] == 30.54 for c in got["configs"].values())
