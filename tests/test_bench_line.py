"""The result line of bench.py stays short enough to be read back whole from the
end of a log: tables go into it as a few numbers per call."""
import json

import bench


def test_tables_are_carried_as_a_few_numbers_per_call():
    row = {"ms_min": 0.1234, "ms_cold": 0.1234, "nnz_kept": 123456789, "gflops": 12345.6, "eff_GBps": 12345.6,
           "eff_over_hbm_peak": 1.2345, "min_GBps": 1234.5, "hbm_frac_compulsory": 0.1234, "traffic_GBps": 7654.3,
           "cache_served": True, "ms": 12.3456}
    calls = [dict(row, mode=m, W=W, speedup_vs_full=12.34) for W in (16, 32, 64, 128, 256)
             for m in ("bucket", "fastrand")] + [dict(row, mode="full", W=0, speedup_vs_full=1.0)]
    table = {"workload": "a graph", "N": 1, "calls": calls, "traffic_source": {"file": "x"}}
    short = bench.brief(table)
    assert short["calls"]["fastrand:64"] == [12.3456, 12345.6, 1234.5, 12.34] and len(short["calls"]) == 11
    assert short["workload"] == "a graph" and "traffic_source" not in short
    stages = bench.brief({"stages": [dict(calls[0], F=F) for F in (256, 41)]})["stages"]
    assert list(stages) == ["F=256 bucket:16", "F=41 bucket:16"]
    assert bench.brief({"rows": [1]}) == {"rows": [1]}
    # seven tables of a full sweep, with room for the head of the line
    assert len(json.dumps([short] * 7)) < 6000
