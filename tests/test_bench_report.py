"""The summary of a kernel trace says of the kernel that the trace shows what that kernel did."""
import csv
import json

import bench


def test_eager_summary_counts_the_launches_of_the_timed_passes(tmp_path, capsys):
    """Bracketed one push at a time (32 launches of another kernel), timed in stages: 33 launches to a pass."""
    stats, log = tmp_path / "stats.csv", tmp_path / "bench.log"
    with open(stats, "w", newline="") as f:
        w = csv.DictWriter(f, ["Name", "Calls", "TotalDurationNs", "AverageNs", "MinNs", "MaxNs", "Percentage"])
        w.writeheader()
        for name, calls, avg in (("k_eager_pass<TraitsF32, 8, true, false, false>", 33 * 52, 29000), ("k_eager_pass<TraitsF32, 16, false, false, false>", 32, 34000)):
            w.writerow(dict(Name=name, Calls=calls, TotalDurationNs=calls * avg, AverageNs=avg, MinNs=avg, MaxNs=avg, Percentage=50))
    line = dict(config=dict(workload="cfg3_2d_small_256streams_eager_emission"), steps=50, warmup=2, ms_per_step=0.97,
                roofline=dict(bound="hbm", kernel="eager", unit="GB/s", peak=8000.0, algorithmic_bytes_per_step=33e6, executed_flops_per_step=33e9))
    log.write_text(json.dumps(line) + "\n")
    bench.trace_summary(str(stats), str(log))
    out = capsys.readouterr().out
    assert "launches_per_step 33.0 x trace average = 0.957 ms" in out
    assert "Algorithmic bytes per launch 1000000; executed flops per launch 1000000000" in out
