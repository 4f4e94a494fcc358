"""bench.py's profile summaries on the CPU: of a kernel template's instances in one run, the time and the counters of
the one that took the most time stand together."""
import csv

import bench

SMALL = "void (anonymous namespace)::k_fit_group<16, 1>((anonymous namespace)::Args)"
LARGE = "void (anonymous namespace)::k_fit_group<2, 32>((anonymous namespace)::Args)"
PLAIN = "(anonymous namespace)::k_fit((anonymous namespace)::Args)"


def test_time_and_counters_of_one_instance(tmp_path):
    rows = [{"name": n, "totaldurationns": str(t), "averagens": str(t / c), "calls": str(c)}
            for n, t, c in ((LARGE, 900.0, 2), (SMALL, 500.0, 10), (PLAIN, 100.0, 1))]
    stats, instances = bench._dominant(rows)
    assert stats["k_fit_group"]["name"] == LARGE and stats["k_fit"]["name"] == PLAIN
    with open(tmp_path / "x_counter_collection.csv", "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
        for d, name, value in ((1, SMALL, 7), (2, LARGE, 40), (2, LARGE, 60), (3, LARGE, 300), (4, PLAIN, 5), (5, SMALL, 9)):
            w.writerow([d, name, "FETCH_SIZE", value])
        w.writerow([2, LARGE, "WRITE_SIZE", 1000])
    assert bench._counter_means(str(tmp_path), "FETCH_SIZE", instances) == {"k_fit_group": 200.0, "k_fit": 5.0}
