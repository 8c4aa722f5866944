"""The line that bench.py prints is short enough to be read back from a log's
tail, holds what the contract asks for, and some of every leg."""
from __future__ import annotations

import json

import bench

KERNELS = {"kernel_%d" % i: {"launches": 1234, "ms_per_step": 1.23456, "avg_launch_ms": 0.0123,
                             "GBps_algorithmic": 1234.5, "per_launch": {"items": 12345678, "edges": 12345678}}
           for i in range(12)}
ROOF = {"bound": "hbm", "achieved": 2163.5, "peak": 8000.0, "unit": "GB/s", "frac": 0.2704, "traffic": 6953411015,
        "kernel": "ms_delta_hub", "launches": 2100, "avg_launch_ms": 1.0881,
        "algorithmic_bytes_per_launch": 2354126142, "traffic_source": "profiles/traffic_rmat-22.json",
        "frac_of_measured_copy": 0.4511, "traffic_GBps": 6390.2}
CPU = {"value": 43363231.36313943, "unit": "TEPS", "cores": 1, "kind": "oracle",
       "sample": "first 4 of the 1024 sources, single-threaded C oracle, 5.9 s", "cpu_model": "AMD EPYC 9575F 64-Core Processor"}
PARITY = {"max_rel_err": 1.2345678901234e-15, "zero_exact": True, "pass": True}


def phase():
    return {"offered_qps": 1.234, "achieved_qps": 34.567, "teps": 1.2345e11, "p50_ms": 1234.56, "p99_ms": 2345.67,
            "max_ms": 3456.78, "failed": 0,
            "by_graph": {"graph-%d" % i: {"requests": 40, "largest_sources": 400, "p50_ms": 1234.5, "p99_ms": 2345.6}
                         for i in range(8)}}


def full():
    leg = {"workload": "a workload of some name", "kernels": KERNELS, "roofline": ROOF, "cpu_baseline": CPU,
           "parity": PARITY, "sources": 64, "teps": 1.2345678901e11}
    return {
        "metric": bench.METRIC, "value": 186093413057.64676, "unit": "TEPS", "n_gpus": 1, "steps": 20, "warmup": 5,
        "ms_per_step": 353.0216495500002, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "batched_over_per_source": 14.876543212345, "forward_GBps_algorithmic": 1797.4, "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": "rmat-22 batched BC", "vertices": 4194304, "undirected_edges": 64155277,
                   "nnz": 128310554, "sources": 1024, "batch_width": 64, "graph_seed": 1003, "source_seed": 2003,
                   "levels_max": 9, "topdown_levels": 70, "bottomup_levels": 51, "block_size": 512, "alpha": 4.0,
                   "beta": 24.0, "chunk_levels": 8,
                   "autotuned": {"batch_width": 64, "block_size": 512, "tuning_s": 1.23, "group_ms": 120.1,
                                 "candidates": [{"batch_width": 64, "block_size": 512, "alpha": 4.0,
                                                 "ms_per_source": 0.2834, "accepted": True}] * 20}},
        "device_ms_per_step": 352.123456789, "ms_per_step_kernel_timed": 360.123456789, "graph_launches_per_step": 48,
        "status": 0, "upload_ms": 123.456789, "source_grouping_ms": 12.3, "hbm_copy_GBps_measured": 5123.4,
        "graph_build_s": 12.3456789, "roofline": ROOF, "per_source_path": dict(leg, ms_per_source=5.4321, block_size=256),
        "per_source_legs": {"rmat-20": dict(leg, ms_per_source=0.8123)},
        "road_batched": {"road-4096": dict(leg, ms_per_pass=210.1, engine="blocks")},
        "forward_pass": {"ms_per_step": 180.11, "GBps_algorithmic": 1797.4, "GBps_hbm_counters": 4745.6,
                         "frac_of_peak_hbm_counters": 0.5932},
        "kernels": KERNELS, "cpu_baseline": CPU, "cpu_baseline_parallel": CPU, "parity": dict(PARITY, sources=16),
        "serving": {p: phase() for p in ("burst", "load50", "load80", "load95")},
        "sssp": {w: dict(leg, ms_per_source=3.123, rounds_mean=12.5, entries_scanned_over_nnz=2.1)
                 for w in ("rmat-22", "road-4096")},
        "pagerank": {w: dict(leg, ms_per_iteration=0.6789) for w in ("rmat-22", "road-4096", "rmat-22-directed")},
        "triangles": {"rmat-22": dict(leg, triangles=2052349654, count_ms=6.123, build_ms=12.34)},
        "directed_bc": {"rmat-22": dict(leg, parity={"per_source": PARITY, "batched": PARITY, "all_pass": True},
                                        batched_over_per_source=12.3456, per_source=dict(sources=64, ms_per_source=4.56),
                                        batched_all_sources=dict(sources=1024, ms=345.6, passes=16))},
    }


def test_line_is_short_and_complete():
    line = json.dumps(bench.headline(full()))
    assert len(line) <= 4096, len(line)
    out = json.loads(line)
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline", "parity"):
        assert out[k] == full()[k] or k == "config"
    assert "kernels" not in line and "candidates" not in line and "by_graph" not in line
    assert out["sssp"]["rmat-22"]["ms_per_source"] == 3.123 and out["sssp"]["rmat-22"]["parity"] is True
    assert out["directed_bc"]["rmat-22"]["parity"] is True
    assert out["serving"]["load80"] == {"achieved_qps": 34.567, "p50_ms": 1234.56, "p99_ms": 2345.67, "failed": 0}


def test_skipped_legs_stay_out():
    doc = full()
    for k in ("serving", "sssp", "pagerank", "triangles", "directed_bc", "road_batched", "per_source_legs",
              "per_source_path"):
        doc[k] = None
    out = bench.headline(doc)
    assert not set(out) & {"serving", "sssp", "pagerank", "triangles", "directed_bc", "road_batched"}
