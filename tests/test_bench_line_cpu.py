"""The line that ``python bench.py`` prints: the fields its readers take from it, short enough to be kept whole."""
import json

import bench


def test_headline_is_short_and_complete():
    block = dict(value=1234.567, unit="TFLOP/s", steps=100, warmup=20, ms_per_step=12.34567, dtype="bf16", ms_per_layer=12.34567,
                 parity_max_err_over_rms=0.0123456789012345,
                 config=dict(workload="c2_prefill_up_proj:up_proj", d_in=4096, d_out=11008, tokens=7539, requests=16, adapters_resident=16,
                             adapters_used=10, segments=10, rank_max=64, weight_sets=2, step="lora_plan_device + lora_linear", plan_amortised_over=224),
                 roofline=dict(bound="mfma", achieved=1234.5, peak=2500.0, unit="TFLOP/s", frac=0.4938, frac_of_measured_ceiling=0.7262,
                               traffic=1234567890, traffic_source="x" * 200, kernel="tile_256x256w4", kernel_us=574.123,
                               algorithmic_bytes=123456789012, algorithmic_flops=123456789012345),
                 cpu_baseline=dict(value=0.123456, unit="TFLOP/s", cores=16, kind="oracle", sample="1234 of 7539 rows of the layer, 2 repetition(s), 1.234 s each"),
                 kernels={"shrink": "y" * 3000})
    per_config = [dict(block, index=i) for i in range(5)]
    per_config[3] = {k: v for k, v in dict(per_config[3], ms_per_layer_sum_of_seven=1.23456).items() if k not in ("ms_per_step", "ms_per_layer")}
    detail = dict(metric=bench.METRIC, n_gpus=1, higher_is_better=True, scaling="weak", vs_baseline=None, data="synthetic", per_config=per_config,
                  batch_size_sweep_config1_shape=["z" * 3000])
    line = bench.headline(detail)
    assert "\n" not in line and len(line) < 1700, len(line)
    out = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data",
              "config", "roofline", "cpu_baseline"):
        assert k in out, k
    assert out["value"] == per_config[bench.HEADLINE]["value"]
    assert out["per_config"]["3"][2] == 1.23456
