"""The benchmark's line on standard output: whoever records a run keeps the last
few kB of what it printed, and a line longer than that is lost whole.  The long
tables go to standard error; nothing is in neither."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

CONTRACT = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
            "vs_baseline", "dtype", "data", "config")


def test_line_is_short_and_complete():
    row = {"kernel": "k" * 40, "avg_us": 1.0, "bytes_per_launch": 10 ** 9, "GBps": 1000.0, "timed_in": "t" * 60}
    form = {"form": "f" * 60, "dr_us": 1.0, "kernels": [row] * 3, "trials_us": [1.0] * 5}
    line = {k: "x" for k in CONTRACT}
    line.update(roofline={"kernel": "k", "note": "n" * 300}, per_mass={"-0.25": {"mg_s": 0.0176}}, kernels=[row] * 8,
                fine_dr_summary={"f64_rhs1": {"GBps": 1.0}}, dslash_24x24x24x64={"f%d" % i: form for i in range(12)},
                dslash_32x32x32x64={"f%d" % i: form for i in range(6)},
                batched_24x24x24x64={"-0.25": dict(setup_s=6.0, lockstep_s=0.87, one_at_a_time_s=3.3,
                                                   max_true_rel_res=1e-11, baselines={"b": ["i" * 20] * 40})},
                cpu_baseline=dict(value=1.0, unit="s", cores=2, kind="oracle", sample="s" * 300,
                                  all_threads={"a%d" % i: 1.0 for i in range(30)}, one_thread=None))
    assert len(json.dumps(line)) > 9000
    short, details = bench.split_line(line)
    assert len(json.dumps(short)) < 2000
    assert all(short[k] == line[k] for k in CONTRACT + ("roofline", "per_mass", "fine_dr_summary"))
    assert short["cpu_baseline"]["value"] == 1.0 and "all_threads" not in short["cpu_baseline"]
    assert short["batched_summary"]["-0.25"] == dict(setup_s=6.0, lockstep_s=0.87, one_at_a_time_s=3.3,
                                                     max_true_rel_res=1e-11)
    for k, v in line.items():
        assert short.get(k) == v or details.get(k) == v or (k == "cpu_baseline" and {**short[k], **details[k]} == v), k


def test_line_without_optional_parts():
    line = {k: "x" for k in CONTRACT}
    line.update(kernels=[], dslash_24x24x24x64=None, dslash_32x32x32x64=None, batched_24x24x24x64=None,
                cpu_baseline=None)
    short, details = bench.split_line(line)
    assert short["cpu_baseline"] is None and details["batched_24x24x24x64"] is None
    assert set(short) | set(details) == set(line)


def test_rates_count_an_operand_once():
    """The rate of an apply does not depend on what its launches read twice or write beside the result."""
    vh = 24 ** 3 * 64 // 2
    for prec, nrhs in ((0, 1), (2, 12)):
        plain = bench.apply_rates(prec, nrhs, [0, 0], vh, 2.0)
        moved = bench.apply_rates(prec, nrhs, bench.canonical_bytes(prec, "schur"), vh, 2.0)
        assert plain["GBps"] == moved["GBps"] == round(bench.dr_compulsory_bytes(prec, nrhs) * nrhs * vh / 2e6, 1)
        assert plain["moved_GBps"] == plain["GBps"] < moved["moved_GBps"]
        assert moved["frac_of_8TBps"] == round(moved["GBps"] / bench.PEAK_HBM_GBS, 3)
