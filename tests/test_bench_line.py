"""The line that bench.py prints: one JSON object with the headline's own values, short
enough to be found whole at the end of captured output."""
import json

import pytest

import bench


def _record(sizes):
    value = 123456789.12345678
    row = {"tokens_per_s": 1378123.123456789, "items_per_s": 2459.123456789, "ms_per_pass": value, "kernels": {"k" * 9: {}}}
    return {
        "metric": bench.METRIC, "value": value, "unit": "tokens/s", "n_gpus": 1, "steps": 20, "warmup": 5,
        "ms_per_step": 26.123456789012345, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": "clip_vit_l14_336 encoder, micro-batch of 64 requests (36928 tokens), pack + encode",
                   "micro_batch": 64, "tokens_per_step": 36928, "layers": 24, "hidden": 1024,
                   "parallelism": "single GPU"},
        "images_per_s": value,
        "roofline": {"bound": "mfma", "kernel": "gemm_bf16_async_res_256x256", "achieved": 1139.123456789,
                     "peak": 2500.0, "unit": "TFLOP/s", "frac": 0.45612345678, "traffic": 461123456.789,
                     "traffic_unit": "HBM bytes per launch", "mean_launch_ms": 0.25751234567,
                     "launches_per_step": 48.0},
        "kernels": {"kernel_%d" % i: {"ms_per_step": value} for i in range(20)}, "gemm_attn_mfma_frac": 0.39512345,
        "serving": {"x": [value] * 50}, "capacity": {"curve": [value] * 50},
        "cpu_baseline": {"value": 427.123456, "unit": "tokens/s", "cores": 16, "kind": "oracle", "sample": "s" * 200},
        "workloads": {name: {"pool": 64, "sweep": [dict(row, micro_batch=b) for b in sizes]}
                      for name in ("clip_vit_l14_336", "qwen2vl_vit_image", "qwen2vl_vit_video", "whisper_large_enc")},
    }


@pytest.mark.parametrize("sizes", [(1, 2, 4, 8, 16, 32, 64), tuple(range(1, 65))])
def test_the_line_is_short_and_keeps_the_headline(sizes):
    record = _record(sizes)
    text = bench.headline(record)
    assert len(text) <= 2000 and "\n" not in text
    line = json.loads(text)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                "vs_baseline", "dtype", "data", "config"):
        assert line[key] == record[key], key
    assert line["roofline"]["kernel"] == record["roofline"]["kernel"]
    if len(sizes) < 10:
        assert line["sweep"]["whisper_large_enc"]["16"] == [1378123, 2459.1]
