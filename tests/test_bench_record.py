"""The benchmark's record: one short line with what a reader of the benchmark needs, the rest apart."""
import json

import bench
import workloads

CONTRACT = {"metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
            "vs_baseline", "dtype", "data", "config"}


def test_headline_is_short_and_complete():
    w = workloads.WORKLOADS["mix_bf16_b2e24"]
    out = {"metric": bench.METRIC, "value": 14627436123.4, "unit": "proj/s", "n_gpus": 1, "steps": 20, "warmup": 3,
           "ms_per_step": 1.1469123456789, "fwd_proj_per_s": 23530987654.3, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "f32", "data": "synthetic",
           "config": {"workload": w.name, "B": w.B, "storage": w.storage, "tol": 1e-6, "max_iter": 64,
                      "passes": "fwd+bwd", "desc": w.desc, "buffer_sets": 1},
           "roofline": {"bound": "hbm", "kernel": "newton_fwd", "achieved": 3010.1, "peak": 8000.0, "unit": "GB/s",
                        "frac": 0.3763, "traffic": 2223800000.0,
                        "valu": {"achieved": 24.01, "peak": 39.32, "unit": "T lane-instr/s", "frac": 0.6106,
                                 "counted_lane_instr_per_launch": 17117000000.0}},
           "path_hbm_frac": 0.5267, "kernels": {"newton_fwd": {"avg_ms": 0.713}}, "max_marginal_err": 1.09e-06,
           "newton_steps": {"hist": list(range(41))}, "configs": {"x": [0.0] * 5000}, "buckets": [1] * 1000}
    headline, detail = bench.split_record(out)
    assert len(json.dumps(headline)) <= 1600  # records keep the last 2000 characters of the output
    assert CONTRACT <= set(headline) and {"roofline", "max_marginal_err"} <= set(headline)
    assert set(headline) | set(detail) == set(out) and not set(headline) & set(detail)
