"""The benchmark's result line: the contract's keys, and short enough for the tail of a log."""
import json

import bench
from paper_2509_01229_amd import api
from paper_2509_01229_amd import workloads as WL


def test_result_line_is_short_and_complete():
    point = {"M": 4096, "N": 28672, "K": 28672, "group": 128, "us": 12345.678, "tops": 12345.678, "gbs": 12345.6, "bound": "mfma",
             "frac_of_roofline": 0.1234, "variant": "solo16_pt_m256[2048 rows]+solo16_g2_m256[512 rows]", "us_same_buffer": 1.0}
    roof = {"bound": "mfma", "achieved": 12345.67, "peak": 5033.2, "unit": "TOP/s", "frac": 0.1234, "kernel": point["variant"],
            "traffic": 123456789, "algorithmic_bytes": 123456789, "algorithmic_ops": 123456789012,
            "frac_of_measured_random_operand_mfma": 0.1234, "workload": "l70b_down_M2048_N8192_K28672"}
    out = {"metric": "W4A8 GEMM TOPS and % of HBM / int8-MFMA roofline vs M (1..4096)", "value": 12345.678, "unit": "TOPS",
           "n_gpus": 1, "steps": 100, "warmup": 10, "ms_per_step": 0.12345, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "int8 x uint4->int8, int32 accumulate, fp16 out", "data": "synthetic",
           "config": {"workload": "prefill_M4096_N8192_K8192", "M": 4096, "N": 8192, "K": 8192, "group": 64, "weight_copies_rotated": 16},
           "roofline": roof, "roofline_hbm": roof, "curve_N8192_K8192": [point] * 13, "curve_N4096_K4096": [point] * 13,
           "calibration": {"stream_read_gbs": 12345.6, "stream_read_gbs_120MiB_launches": 12345.6, "mfma_i8_constant_tops": 12345.6,
                           "mfma_i8_random_tops": 12345.6, "note": "x" * 300},
           "configs": [point] * 23, "activation_quant": [point] * 3, "reference_w8a8_own": [point] * 3, "ablation_dequant": point,
           "mfma_shape": point, "grouped_moe": [point] * 6,
           "cpu_baseline": {"value": 0.123456, "unit": "TOPS", "cores": 16, "kind": "oracle", "sample": "x" * 150}}
    line = bench.short_line(out)
    contract = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline",
                "dtype", "data", "config")
    assert all(line[k] == out[k] for k in contract)
    assert line["curve_N8192_K8192"][0] == [4096, 12345.678, 0.1234]
    assert len(json.dumps(line)) < 1950


def test_traffic_is_that_of_the_kernels_that_run():
    """The result line's two kernels have a measured traffic under the names that the library reports for them."""
    for name in ("prefill_M4096_N8192_K8192", bench.HBM_WORKLOAD):
        s = WL.by_name(name)
        kernel = api.w4a8_describe_launch(s.M, s.N, s.K, s.group)[0]
        traffic = bench.measured_traffic(name, kernel)
        assert traffic and traffic >= bench.algorithmic_bytes(s.M, s.N, s.K, s.group), kernel
