"""The line that bench.py prints on stdout fits the 2000 characters that a log keeps of a run's end, with every field of the
headline in it; the whole record goes to stderr."""
import json

import bench

HEAD = {"metric": "sliced block-forward TFLOP/s (% MFMA peak) + peak live activation bytes vs unsliced", "value": 900.1234567890123,
        "unit": "TFLOP/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 10.123456789012345, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic"}


def test_line_is_short_and_whole(capsys):
    live = {"sliced": 12345678901, "unsliced_same_kernels": 123456789012, "ratio": 0.12345678901234567, "workspace_bytes": 1 << 35}
    stages = {f"stage_{i}": {"avg_us": 123.45, "launches_per_step": 25.0, "ms_per_step": 3.0863} for i in range(20)}
    roof = {"bound": "mfma", "kernel": "conv3x3 (conv1 + conv2 launches)", "achieved": 1012.123456789012, "peak": 2500.0, "unit": "TFLOP/s",
            "frac": 0.40484938271560, "traffic": {"text": "x" * 900}, "avg_launch_us": 212.12345678901234, "algorithmic_flop_per_launch": 217432719360.0}
    one = {"TFLOP/s": 900.1234567890123, "ms_per_step": 10.123456789012345, "live_activation_bytes": live, "per_block": stages, "roofline": roof}
    record = dict(HEAD, config={"workload": "w" * 400, "algorithmic_flop_per_step": 9043214567890.0, "tokens": 460800},
                  frac_mfma_peak=0.3712345678901234, ms_reps=[1.2345678901234567] * 50, live_activation_bytes=live, memory_check=stages,
                  hbm_floor_check=stages, rehash={"cos": 0.99, "decision": 1}, roofline=roof, per_block=stages, stages=stages,
                  kernel_source_hash="0123456789abcdef", configs={f"cfg{i}s": one for i in range(7)},
                  cpu_baseline={"value": 0.0786075403511966, "unit": "TFLOP/s", "cores": 16, "kind": "oracle", "sample": "y" * 300})
    bench.emit(record)
    out, err = capsys.readouterr()
    assert json.loads(err) == record
    assert out.count("\n") == 1 and len(out) < 2000, len(out)
    line = json.loads(out)
    for k in (*HEAD, "config", "frac_mfma_peak", "kernel_source_hash"):
        assert line[k] == record[k]
    assert line["live_activation_bytes"]["ratio"] == live["ratio"] and line["roofline"]["achieved"] == roof["achieved"]
    assert set(line["configs"]) == set(record["configs"]) and line["cpu_baseline"]["value"] == record["cpu_baseline"]["value"]
