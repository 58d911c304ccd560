"""bench.py's line on stdout: short enough for a log's tail to hold it whole, the
keys of its contract in it, whatever legs ran.  The record here has the shape and
the number lengths of a full run."""
import json

import bench

X = 12345678901.123456


def record():
    legs = lambda names, v: {n: json.loads(json.dumps(v)) for n in names}  # noqa: E731
    q = {"us_per_call": X, "tracks_per_s": X, "GB_s": X, "bound": "hbm", "frac_alu": X, "frac_hbm": X, "frac": X,
         "ops_per_track": X, "bytes_per_track": 73}
    solid = dict(legs(("inside", "safety", "dist_in", "dist_out", "fused"), q), separate_vs_fused_time=X,
                 walk_counts={"fused": [1 << 24] * 5})
    load = {"offered_baskets_per_s": X, "achieved_track_queries_per_s": X, "p50_ms": X, "p99_ms": X, "max_ms": X, "load": 0.95}
    point = {"saturation": {"baskets_per_s": X}, "loads": [load] * 3, "rounds": 9999, "largest_round": 64,
             "serial": {"saturation": {"baskets_per_s": X}, "loads": [load] * 3, "batching_speedup": X}}
    return {
        "metric": "track-steps/s", "value": X, "unit": "track-steps/s", "n_gpus": 1, "steps": 20, "warmup": 5,
        "ms_per_step": X, "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": "w" * 80, "tracks": 1 << 20, "track_steps": 70324084, "max_steps": 128,
                   "steps_world_layer_module": [1 << 24] * 3},
        "roofline": {"bound": "alu", "kernel": "k_lane_transport", "achieved": X, "peak": X, "unit": "u" * 90, "frac": X,
                     "traffic": X, "ops_per_transport": X, "ops_per_launch": X, "launches_per_transport": X,
                     "avg_launch_ms": X, "kernel_ms_per_transport": X, "algorithmic_bytes_per_transport": 1 << 30,
                     "frac_measured_fp64_roof": X, "hbm": legs("abcdef", X), "accounting": "a" * 400},
        "roofs": {"hbm_triad_GBs": X, "hbm_copy_GBs": X, "fp64_fma_Tlane_ops": X, "fp64_TFLOPs": X,
                  "nominal": {"hbm_GBs": X}, "method": "m" * 120},
        "tuning": legs(("step_grid scatter_grid cell_bits solid_block solid_grid step_waves transport sort_bits sort_key "
                        "lane_waves lane_stage lane_grid lane_sched").split(), 1024),
        "work": legs("abcdefghijkl", [1 << 30] * 2), "wall_s": X, "flags_nonzero": 0,
        "cpu_baseline": {"value": X, "unit": "track-steps/s", "cores": 16, "kind": "oracle", "sample": "s" * 80},
        "oracle_parity": {"tracks": 1 << 20, "track_steps": 70324084, "mismatched_tracks": 0, "sequence_mismatches": 0,
                          "flagged_tracks": 0, "flagged_first": list(range(1 << 20, (1 << 20) + 20)),
                          "flagged_that_differ": 0, "max_step_err_mm": X, "bar": "b" * 100},
        "fp32_refine": {"ms_per_step": X, "value": X, "identical_to_fp64": True, "fp32_screened_frac": X,
                        "oracle_parity": {"bar": "b" * 100}},
        "physics_limited": legs(("shortcut", "no_shortcut"), {"ms_per_step": X, "track_steps_per_s": X, "track_steps": 1 << 27,
                                                              "physics_limited_steps": 1 << 24, "shortcut_steps": 1 << 24}),
        "serving": {"slots": 64, "points": [dict(point, precision="fp64"), dict(point, precision="fp32_refine")]},
        "solids": legs(("box", "tubs", "cons", "sphere", "trd", "pcon"), solid),
        "protocol": legs(("box", "tubs"), [{"n": 1 << 20, "us_per_call": X, "tracks_per_s": X}] * 9),
        "cpu_baseline_solids": legs("abcdef", [q] * 9),
        "composites": {"solids": legs([f"composite_name_{i}" for i in range(8)], {"fused_us_per_call": X, "tracks_per_s": X}),
                       "transport": {"tracks": 1 << 20, "ms_per_call": X, "track_steps_per_s": X}},
    }


def test_line_holds_the_contract_and_fits():
    res = record()
    line = json.dumps(bench.summary(res))
    assert len(line) <= bench.LINE_MAX and "\n" not in line
    got = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config"):
        assert got[k] == res[k]
    assert len(json.dumps(res)) > 2 * bench.LINE_MAX  # what used to be the line


def test_line_without_the_other_legs():
    res = {k: v for k, v in record().items() if k not in ("roofs", "fp32_refine", "physics_limited", "serving", "solids",
                                                          "protocol", "cpu_baseline_solids", "composites")}
    assert json.loads(json.dumps(bench.summary(dict(res, roofs=None))))["roofline"]["kernel"] == "k_lane_transport"
