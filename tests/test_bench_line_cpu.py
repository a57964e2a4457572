"""The line that bench.py prints: what it says of the other workloads stays short, whatever a run measured of them."""
import json

import bench


def full(name):
    classes = {c: {"ms_per_step": 9.263444667682052, "launches_per_step": 129, "tflops": 925.3613110502813,
                   "frac_mfma_peak": 0.37014452442011253, "gbs": 1710.232482228906, "frac_hbm_peak": 0.21377906027861326}
               for c in ("gemm", "attention", "realign", "deviation", "topk", "norm", "other", "finish")}
    return {"workload": name, "ratio": 0.15, "schedule": "gradual", "ttft_ms": 12.159220000000914, "kernel_classes": classes,
            "hkvd_token_layers_per_s": 1546698.3903867172, "launches_per_step": 300, "roofline": {"achieved": 1.0}}


def test_other_workloads_are_summarised():
    rows = [bench.summary(full(f"yi34b-r0.15-int8-{i}")) for i in range(len(bench.EXTRA))]
    assert rows[0] == {"workload": "yi34b-r0.15-int8-0", "ratio": 0.15, "ttft_ms": 12.1592, "launches_per_step": 300,
                       "hkvd_token_layers_per_s": 1546700.0, "gemm_tflops": 925.361, "attention_tflops": 925.361}
    assert len(json.dumps(rows)) < 2000
    no_profile = {k: v for k, v in full("tiny").items() if k not in ("kernel_classes", "launches_per_step")}
    assert "gemm_tflops" not in bench.summary(no_profile)


def test_short_keeps_everything_but_digits():
    v = {"a": [1.23456789, 7, "x", None], "b": {"c": True, "d": float("inf")}}
    assert bench.short(v) == {"a": [1.23457, 7, "x", None], "b": {"c": True, "d": float("inf")}}
