"""The line that bench.py prints: the figures a reader needs, short enough to survive in the tail of a log."""
import json

import bench


def measured(kernels):
    """A result of one configuration with every part that bench.py can measure."""
    ent = dict(bound="mfma", mfma_dtype="bf16", ms_per_step=123.4567, launches_per_step=1234, avg_launch_ms=0.12345,
               executed_flops_per_launch=333989237996.3077, achieved=1867.11, peak=2500.0, unit="TFLOP/s", frac=0.7468,
               definition_equiv_tflops=344.52)
    part = dict(bound="hbm", kernel="syrk_reduce_kernel", achieved=1534.6, peak=8000.0, unit="GB/s", frac=0.1918,
                ms_per_step=2.7573, launches_per_step=5, algorithmic_bytes_per_step=4231398528, moved_gbps=3123.5, note="n" * 300)
    return dict(ms_per_step=123.4567, cold_ms_per_step=123.4567, cold_note="n" * 200, dtype="bf16 in, f32 accumulate",
                config=dict(workload="transformer_encoder_bf16", variant="inverse", layers=144, batch=64, damping=0.003, decay=0.95,
                            in_dtype="bf16", gout_sigma=0.03162),
                stage_ms={f"some_stage_{i}": 12.3456 for i in range(21)}, launches_per_step={f"some_stage_{i}": 1234 for i in range(21)},
                roofline=dict(ent, kernel="gemm_split_kernel", traffic=147179262, share_of_step=0.378, note="n" * 300),
                kernels={k: dict(ent, note="n" * 100) for k in kernels},
                kf_gemm=dict(mfma_util_pct=22.91, ms_per_step=7.5661, definition_equiv_tflops=572.68, note="n" * 300),
                algorithmic_work={f"part_{i}": 2167382605824 for i in range(8)},
                stale_schedule=dict(update_factors_ms=7.3971, invert_ms=39.7506, precondition_ms=10.7201, F_freq=50, K_freq=500,
                                    amortised_ms_per_iteration=10.9475),
                running_average=part, im2col=dict(part, counter_bytes_per_launch=179227000),
                cpu_baseline=dict(value=465406.0, unit="ms", cores=16, kind="oracle", sample="n" * 200), steps=5)


def test_printed_line_is_short_and_keeps_the_contract():
    kernels = [c[0] for c in bench.CLASSES.values()]
    head = measured(kernels)
    out = dict(head, metric=bench.METRIC, value=head["ms_per_step"], unit="ms", n_gpus=1, steps=20, warmup=5,
               higher_is_better=False, scaling="weak", vs_baseline=None, data="synthetic", kf_gemm_mfma_util_pct=22.91,
               other_configs={name: measured(kernels) for name in bench.OTHERS})
    text = json.dumps(bench.printed(out))
    assert len(text) < 6000
    line = json.loads(text)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
              "dtype", "data", "config", "cold_ms_per_step", "kf_gemm_mfma_util_pct"):
        assert line[k] == out[k]
    for k in ("kernel", "bound", "achieved", "peak", "unit", "frac", "traffic"):
        assert line["roofline"][k] == out["roofline"][k]
    assert line["cpu_baseline"]["value"] == out["cpu_baseline"]["value"]
    assert set(line["kernels"]) == set(kernels)
    assert set(line["other_configs"]) == set(bench.OTHERS)
    assert all(o["ms_per_step"] == 123.4567 for o in line["other_configs"].values())
