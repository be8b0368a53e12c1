"""The benchmark's stdout line: the contract's keys, and short enough to be kept whole by a reader that keeps 8 KB of a program's
output.  Parity unpinned (own benchmark)."""
import json

import bench


def test_line_is_short_and_complete():
    route = "quant_act (+ group row sums) + group-bias pre-pass + prefill per-tile tile=128x256 waves=8 ring=3 ksplit=16 mode=5 grid=65535 + k-split reduce"
    roof = {"bound": "mfma", "achieved": 3118.6, "peak": 5033.0, "unit": "TOP/s", "frac": 0.6196, "kernel": route, "kernel_us": 616.984,
            "algorithmic_bytes": 385949696, "target": {"frac": 0.6, "of": "mfma", "met": True}, "traffic": 1174624944}
    point = {"variant": "perchannel", "M": 4096, "K": 8192, "N": 28672, "steps": 100, "replays": 5, "weight_copies_rotated": 47, "hip_graph": True,
             "ms_per_step": 0.634567, "ms_per_step_min": 0.634567, "ms_per_step_max": 0.634567, "step_route": route, "gemm_route": route,
             "gemm_us": 616.984, "gemm_us_min": 616.984, "gemm_us_max": 616.984, "quant_act_us": 17.706, "quant_act_gbs": 5912.3, "tops": 3032.123,
             "roofline": roof, "mfma_util": None, "oracle": {"seconds": 12.345, "rows": 443, "gmac_per_s": 36.79, "extrapolated": True}}
    names = list(bench.SWEEP)
    out = {"metric": bench.METRIC, "value": 3032.123, "unit": "TOPS", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 0.634567,
           "ms_per_step_min": 0.634567, "ms_per_step_max": 0.634567, "replays": 5, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "int8", "data": "synthetic", "config": {"workload": names[0], "step": route, "group": 128},
           "roofline": roof, "clocks": {"source": "x" * 200}, "sweep": [dict(point, workload=n) for n in names],
           "targets": {"met": len(names), "of": len(names), "met_workloads": names},
           "real_valued_group_scale": [{"shape_of": n, "entry": "qqq_gemm_w4a8_pergroup_f16scale", "roofline": {"frac": 0.5}} for n in names[:2]],
           "weight_front_end": [{"layer": "a layer", "N": 28672, "K": 8192, "kernel": "quant_weight_kernel (perchannel)", "us": 105.5, "bound": "hbm",
                                 "achieved_gbs": 5568.4, "frac": 0.696}] * 6,
           "offline_stage": [{"call": "qqq_gptq_quantize_w4_perchannel", "K": 1024, "N": 4096, "ms": 0.747}] * 4,
           "cpu_baseline": {"value": 1.0, "unit": "TOPS", "cores": 16, "kind": "oracle", "sample": "x" * 300,
                            "per_workload": {n: point["oracle"] for n in names}}}
    text = json.dumps(bench.stdout_line(out))
    assert len(json.dumps(out)) > 10000 and len(text) < 8000, len(text)
    line = json.loads(text)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype",
                "data", "config"):
        assert line[key] == out[key], key
    assert [l["workload"] for l in line["sweep"]] == names and "per_workload" in out["cpu_baseline"]
