"""bench.py's printed line: short enough to be read whole from the end of an output, with the headline exact."""
import json

import bench


def test_line_is_short_and_keeps_the_headline():
    kernels = [{"kernel": "gemm_bf16_crew_kernel<256, 256, 2, 4, true, false, float, false>%d" % i, "groups": 256, "launches_per_step": 1.0,
                "ms_per_launch": 0.4123456789, "ms_per_step": 0.4123456789, "flops_per_launch": 1.23456789e12,
                "bytes_per_launch": 1.23456789e9} for i in range(9)]
    calls = {c: {"ms": 0.123456789012, "tflops": 1234.56789012, "gbs": 1234.56789012, "frac": 0.123456789012}
             for c in ("fwd", "bwd", "bwd_input", "bwd_weight")}
    config = {"ms_per_step": 0.123456789012, "ms_per_step_batches": [0.123456789012] * 5, "ms_per_step_warm": 0.123456789012,
              "tokens": 16384, "in": 4096, "out": 11008, "l": 8, "k": 256, "R": 2048, "dtype": "bf16", "per_call": calls,
              "bound": "mfma", "step_frac": 0.123456789012, "step_frac_of_measured": 0.123456789012, "tflops": 1234.56789012,
              "tokens_per_s": 12345678.9012345, "three_call_ms_per_step": 0.123456789012, "kernels": kernels[:6],
              "dense_context": {"ms_per_step": 0.123456789012, "kind": "k" * 80, "tflops": 1234.56789012,
                                "sketched_over_dense_time": 0.123456789012, "sketched_over_dense_flops": 1.0}}
    out = {"metric": "m" * 70, "value": 6646543.123456789, "unit": "tokens/s", "n_gpus": 1, "steps": 20, "warmup": 5,
           "ms_per_step": 2.4650123456789, "config": {"workload": "c4_llm_mlp", "calls_per_step": ["fwd", "bwd"], "timing": "t" * 40,
                                                      "cache": "c" * 60},
           "ms_per_step_batches": [2.46501234567] * 5, "per_call": calls, "roofline": {"achieved": 1234.56789012, "how": "h" * 120,
                                                                                     "kernel": kernels[0]["kernel"]},
           "kernels": kernels, "configs": {"c%d_bert_base_ffn_up" % i: config for i in range(8)},
           "measured_peak": {"a%d" % i: 1234.56789012 for i in range(12)},
           "cpu_baseline": {"value": 1234.56789012, "unit": "tokens/s", "cores": 16, "kind": "oracle", "sample": "s" * 120}}
    line = json.dumps(bench.summary(out))
    assert len(line) < 6000 and "\n" not in line, len(line)
    back = json.loads(line)
    assert back["value"] == out["value"] and back["ms_per_step"] == out["ms_per_step"]
    assert set(back["configs"]) == set(out["configs"]) and back["configs"]["c0_bert_base_ffn_up"]["ms_per_step"] == 0.12346
