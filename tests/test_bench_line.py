"""bench.py's one JSON line: complete, and short enough for readers that keep only the last 16000 characters of the output."""
import json
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench


def record(n_kernels):
    v = 1234.567890123456
    modes = {"sequential": v, "stream_parallel": v, "regulated": v}
    return {
        "workload": "tenant mix of the evaluation (Table 2): resnet50(16)+vgg16(8)+mobilenetv3-large(32) bf16 224x224", "items_per_round": 56,
        "tenants": ["resnet50(16)", "vgg16(8)", "mobilenetv3_large(32)", "bert_base(8)"], "dtype": "bf16", "plan": "unsplit+refined(14 ops decomposed)",
        "plan_kind": "stream-parallel (the plan holds no decomposition and no pointers)", "issue_threads": False, "launches_per_round": 377,
        "ms_per_step": v, "regulated_images_per_s": v, "sequential_images_per_s": v, "stream_parallel_images_per_s": v, "speedup_vs_sequential": v,
        "speedup_vs_stream_parallel": v, "makespan_ms_median": modes, "makespan_ms_p10_p90": {k: [v, v] for k in modes}, "mfma_frac_of_peak": modes,
        "plan_selection": {"profile_s": v, "search_s": v, "refine_s": v, "trial_ms": {f"candidate-{i}": v for i in range(12)},
                           "model_vs_measured": {f"candidate-{i}": {"model": modes, "measured_ms": v} for i in range(12)}},
        "kernels": {f"igemm_dma_taps_bf16_128x128x{i}": {"launches": 26, "ms_per_round": v, "TFLOP/s": v, "GB/s": v} for i in range(n_kernels)},
        "roofline": {"kernel": "igemm_dma_taps_f32_64x64x32s3", "bound": "mfma", "achieved": v, "peak": v, "frac": v, "share_of_kernel_time": v,
                     "duration_basis": "x" * 200, "launches_per_round": 16, "traffic": None},
        "cpu_baseline": {"value": v, "note": "x" * 300},
    }


def test_the_line_is_one_short_line_that_names_every_workload():
    text = bench.line(record(20), 20, 5, {c: record(20) for c in (3, 4, 5)}, {c: record(20) for c in (6, 7, 8)})
    assert "\n" not in text and len(text) < 12000, len(text)
    out = json.loads(text)
    assert {"metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data",
            "config", "roofline", "cpu_baseline", "kernels"} <= set(out)
    assert out["steps"] == 20 and out["warmup"] == 5 and out["value"] == 1234.57 and out["config"]["launches_per_round"] == 377
    assert set(out["per_config"]) == {"3", "4", "5"} and set(out["paper_mixes"]) == {"6", "7", "8"}
    assert out["per_config"]["4"]["roofline"]["kernel"].startswith("igemm_dma") and out["paper_mixes"]["8"]["mfma_frac_of_peak"] == 1234.57
