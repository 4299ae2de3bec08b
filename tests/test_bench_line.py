"""The line that bench.py prints: short enough to be recorded whole, with every field a reader of it needs."""
import json

import bench


def _out(n_workloads, n_fractions):
    entry = lambda i: dict(r="%d/100" % i, k=[1100 + i, 409], ms=1.23456 + i, tflops=1234.5, dx_ms=1.16407, dw_ms=0.17805,
                           prep_ms=0.04245, finish_ms=0.02454, layers=[dict(name="up", k=110, ms=0.5967, tflops=1250.4)] * 2,
                           speedup_vs_full=1.9770 - i / 100, ideal_speedup=1.9804, over_r0_ms=0.08091, over_r0_us_per_channel=0.5394)
    kernels = [dict(kernel="quant_act", ms=0.13554, launches=2.0, gflop=1477.469, mbytes=634.126, bound="hbm", roof_ms=0.07927,
                    frac=0.5848, gbps=4678.4)] * 7
    block = dict(workload="cfg3: qkv T=12288 768->2304, out T=12288 768->768, ffn1 T=12288 768->3072, ffn2 T=12288 3072->768, "
                          "r=1/4, W8A8, dY channel-major", k=[576, 192, 768, 192], step_ms=0.52683, tflops=412.7,
                 dx_frac_of_mfma_peak=0.2512, kernels=kernels, products_per_layer=[dict(layer="up", dx=kernels[0], dw=kernels[0])] * 4,
                 sweep=[entry(i) for i in range(n_fractions)])
    roofline = dict(bound="mfma", achieved=1268.0786621959005, peak=2500.0, unit="TFLOP/s", frac=0.5072314648783602,
                    traffic=1248848938.0, kernel="k_gemm_dx8", avg_kernel_ms=0.58, kernels=kernels,
                    products_per_layer=block["products_per_layer"][:2], sweep=[entry(i) for i in range(n_fractions)],
                    variants=dict(r="1/4", selected_idx_ms=1.62), extras={"bias_grad": dict(ms=0.045, note="x" * 300)},
                    workloads=[block] * n_workloads)
    return dict(metric="m", value=998.4, unit="TFLOP/s", n_gpus=1, steps=20, warmup=5, ms_per_step=1.85, higher_is_better=True,
                scaling="weak", vs_baseline=None, dtype="bf16", data="synthetic", config=dict(workload="w" * 200), roofline=roofline,
                cpu_baseline=dict(value=0.49, kind="oracle"))


def test_line_is_short_and_whole():
    out = _out(9, 8)
    text = bench.output_line(out)
    assert len(text) <= bench.MAX_LINE and "\n" not in text
    line = json.loads(text)
    for n in out:
        if n != "roofline":
            assert line[n] == out[n], n
    assert line["roofline"]["frac"] == out["roofline"]["frac"] and line["roofline"]["kernels"] == out["roofline"]["kernels"]
    assert [e["speedup_vs_full"] for e in line["roofline"]["sweep"]] == [e["speedup_vs_full"] for e in out["roofline"]["sweep"]]
    assert len(line["roofline"]["workloads"]) == 9 and line["roofline"]["workloads"][0]["speedup_vs_full"]["7/100"] == 1.907
    assert "layers" in out["roofline"]["sweep"][0] and "note" in out["roofline"]["extras"]["bias_grad"]      # left as it was


def test_line_that_would_be_too_long_loses_parts_of_the_roofline():
    text = bench.output_line(_out(60, 60))
    assert len(text) <= bench.MAX_LINE
    line = json.loads(text)
    assert line["value"] == 998.4 and line["roofline"]["achieved"] > 0 and line["cpu_baseline"]["kind"] == "oracle"
