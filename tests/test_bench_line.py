"""The benchmark's stdout line: the contract's keys, short enough to be kept whole
where only the last 2000 characters of the output are."""
import json

import bench


def _record(surrogate):
    rates = lambda names: {n: dict(mlups=123456.7, ms_per_step=0.12345, hbm_frac=0.1234) for n in names}
    return dict(
        metric=bench.METRIC, value=123456.7, unit="MLUPS", n_gpus=1, steps=20, warmup=5, ms_per_step=0.12345,
        higher_is_better=True, scaling="weak", vs_baseline=None, dtype="f32", data="synthetic",
        config=dict(workload="rayleigh_taylor_128x512x128 rayleigh-taylor At=0.5 Re=256 W=4 c=0.997",
                    grid=[128, 512, 128], nodes=8388608, storage="fp16", walls="y", parallelism="single-gpu"),
        roofline=dict(bound="hbm", achieved=1234.5, peak=8000.0, unit="GB/s", frac=0.1234, traffic=1366828148.0,
                      algorithmic_bytes_per_step=1342177280, kernel="x" * 90, copy_gbs=6417.3, frac_of_copy=0.7076,
                      copy_probe={str(k): 1.0 for k in range(40)}),
        secondary=rates(["bf16", "fp32", "fp16+fd", "fp16+q27"]),
        checks={m: dict(finite=True, sum_phi=1.0, umax=0.1) for m in ("fp16", "bf16", "fp32")},
        workloads=rates(["static_droplet_32_fp64", "static_droplet_32_fp16", "rising_bubble_128x128x256_fp16",
                         "rising_bubble_128x128x256_fp32", "taylor_green_256_fp16", "taylor_green_256_fp32"]),
        horizons={str(k): [0.1] * 500 for k in range(10)},
        cpu_baseline=dict(value=18.923, unit="MLUPS", cores=16, kind="oracle", cpu_model="m" * 60, sample="s" * 80),
        surrogate=surrogate)


def test_line_is_short_and_whole():
    full = dict(runs={str(k): dict(seconds=0.1) for k in range(200)}, coupling=dict(push_ms=1.23456789),
                unet_roofline=dict(forward_ms=0.4588949203491211, frac=0.2592179856615138,
                                   train_step_ms=1.6055740356445312),
                lowest_error_schedule=dict(schedule="s", phi_l2_error=0.006994869726171839, speedup=1.0125823563891652))
    full["speedup_at_err_1e-2"] = 1.0197793046827883
    for sur in (full, {"error": "RuntimeError: " + "e" * 5000}):
        rec = _record(sur)
        line = json.dumps(bench.summary(rec))
        assert len(line) < 1950 and "\n" not in line
        got = json.loads(line)
        for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
                  "vs_baseline", "dtype", "data", "config"):
            assert got[k] == rec[k]
        assert got["roofline"]["frac"] == rec["roofline"]["frac"] and got["finite"] is True


def test_line_without_the_optional_parts():
    rec = _record({})
    for k in ("workloads", "horizons", "cpu_baseline", "surrogate"):
        del rec[k]
    got = bench.summary(rec)
    assert "surrogate" not in got and "cpu_baseline" not in got and got["value"] == rec["value"]
