"""The line bench.py prints: what it has to hold, and short enough that the end of the output,
2,000 characters, holds all of it."""
import json

import bench


def config(name):
    times = dict(median_us=12345.678901234567, mean_us=12345.678901234567, back_to_back_us=12345.678901234567)
    return dict(workload=name, best=times, sequential=times, best_mode="multi_stream_graph", zero_copy_concat=True,
                roofline=dict(kernel="igemm_f16_tile128x128_tail", bound="mfma", achieved=1234.5678901234567, peak=2500.0, unit="TFLOP/s",
                              frac=0.12345678901234567, traffic=123456789012, launches_per_step=123, avg_launch_us=123.45678901234567,
                              flops_per_launch=1e12 / 3, bytes_per_launch=1e9 / 3),
                roofline_fraction=0.12345678901234567,
                **{"speedup_" + k: 1.2345678901234567 for k in ("multi_stream_graph", "persistent", "chained", "fused")})


def test_the_line_is_short_and_complete():
    configs = [config(n) for n in ("googlenet_like", "inception_block", "inception_v3_like", "bert_base_like", "random_wide_dag", "nasnet_like")]
    cpu = dict(value=123456.78901234567, unit="us", cores=16, kind="oracle", one_thread_us=123456.78901234567,
               sample="123 full pass(es) of the googlenet_like DAG (numpy fp64, all 81 operators), median",
               timed_executor_matches_oracle=dict(executor="multi_stream_graph", sinks=1, max_abs_err=5.9604644775390625e-08, within_tolerance=True))
    line = bench.result_line(1000, 50, configs[0], configs[1:], cpu)
    assert {"metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data",
            "config", "roofline", "cpu_baseline"} <= set(line)
    assert line["value"] == 12345.68 and line["ms_per_step"] == 12.34568
    assert len(json.dumps(line)) < 1950
