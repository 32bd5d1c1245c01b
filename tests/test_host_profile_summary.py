"""paper_2511_10333_amd/profile_summary.py on small hand-made rocprofv3 CSVs: the calibration factor,
the per-launch means, the kernel-name folding and the line bench.py reads must come out as computed
by hand."""
import csv
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = ["Correlation_Id", "Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"]


def _write(folder, rows):
    os.makedirs(folder, exist_ok=True)
    with open(os.path.join(folder, "c_counter_collection.csv"), "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(HEAD)
        for i, (kernel, counter, value) in enumerate(rows):
            w.writerow([i, kernel[1], kernel[0], counter, value])


def test_traffic_summary_scales_by_the_copy_calibration(tmp_path):
    copy = ("copy_kernel(float*)", 1)
    # a 1 GiB copy that FETCH_SIZE reads as 524288 KiB (two bytes per counted byte) and WRITE_SIZE as 1048576
    _write(tmp_path / "cal_f", [(copy, "FETCH_SIZE", 524288.0)])
    _write(tmp_path / "cal_w", [(copy, "WRITE_SIZE", 1048576.0)])
    full = "void edgc::k_pass_p_deferred_full<1, 4, true, false, 8>(edgc::Group)"
    # two launches; the second one's counter arrives in two rows (two shader engines): summed per dispatch
    _write(tmp_path / "f", [((full, 1), "FETCH_SIZE", 1000.0), ((full, 2), "FETCH_SIZE", 500.0),
                            ((full, 2), "FETCH_SIZE", 1500.0), (("void edgc::k_chol(edgc::Group, unsigned int)", 3), "FETCH_SIZE", 10.0)])
    _write(tmp_path / "w", [((full, 1), "WRITE_SIZE", 300.0), ((full, 2), "WRITE_SIZE", 500.0)])
    out = tmp_path / "t.md"
    r = subprocess.run([sys.executable, "-m", "paper_2511_10333_amd.profile_summary", "traffic", "--workload", "w", "--rank", "8",
                        "--fetch", str(tmp_path / "f"), "--write", str(tmp_path / "w"), "--cal-fetch", str(tmp_path / "cal_f"),
                        "--cal-write", str(tmp_path / "cal_w"), "--out", str(out)], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    text = out.read_text()
    # mean fetch = (1000 + 2000) / 2 = 1500 KiB x 2, mean write = 400 KiB x 1 -> 3400 KiB
    want = 3400 * 1024
    line = [l for l in text.splitlines() if l.startswith("traffic_bytes_per_launch k_pass_p_deferred ")]
    assert len(line) == 1 and abs(float(line[0].split()[-1]) - want) < 1.0     # the whole-tile kernel under the pass's name
    assert "traffic_bytes_per_launch k_chol 2.048000e+04" in text               # 10 KiB x 2, no writes counted

    sys.path.insert(0, ROOT)
    import bench
    (tmp_path / "traffic_probe_r8.md").write_text(text)
    got = bench.traffic_from_profile("probe", 8, "k_pass_p_deferred", folder=str(tmp_path))
    assert got[0] == want


def test_counters_summary_separates_launches_that_did_nothing(tmp_path):
    k = "void edgc::k_hist<float, 4, 1024>(edgc::EntGroup)"
    _write(tmp_path / "c", [((k, 1), "FETCH_SIZE", 1000.0), ((k, 2), "FETCH_SIZE", 2.0), ((k, 3), "FETCH_SIZE", 3000.0)])
    out = tmp_path / "c.md"
    r = subprocess.run([sys.executable, "-m", "paper_2511_10333_amd.profile_summary", "counters", "--dir", str(tmp_path / "c"),
                        "--title", "t", "--out", str(out)], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    row = [l for l in out.read_text().splitlines() if l.startswith("| `k_hist<float, 4, 1024>`")]
    assert row == ["| `k_hist<float, 4, 1024>` | 2 | 1 | 2000 |"]      # two live launches, one idle, mean of the live ones


def test_cells_summary_lists_every_kernel_however_short(tmp_path):
    import json
    cell = {"dtype": "f32", "stride": 1000, "bins": 256, "n_sampled": 10, "ms": 0.02, "reads_of_sample": 2, "sample_gbs": 1.0,
            "gradient_gbs": 2.0, "kernels": {"k_minmax": {"avg_us": 3.9}, "k_hist": {"avg_us": 10.3}}}
    (tmp_path / "c.json").write_text(json.dumps({"cells": [cell]}) + "\n")
    out = tmp_path / "c.md"
    r = subprocess.run([sys.executable, "-m", "paper_2511_10333_amd.profile_summary", "cells", "--json", str(tmp_path / "c.json"),
                        "--title", "t", "--out", str(out)], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    assert "| f32 | 1000 | 256 | 10 | 0.0200 | 2 | 1 | 2 | `k_minmax` 3.9, `k_hist` 10.3 |" in out.read_text()


def test_reads_of_a_sample_follow_from_the_kernels_however_short_they_are():
    sys.path.insert(0, ROOT)
    from bench_entropy import reads_of_sample
    short = {"avg_us": 2.0, "gbs": 1.0}
    assert reads_of_sample({"k_minmax": short, "k_hist": short}, 4096) == 2
    assert reads_of_sample({"k_minmax": short, "k_hist": short}, 65536) == 3
    assert reads_of_sample({"k_minmax": short, "k_wide_hist": short, "k_wide_reduce": short}, 65536) == 2
    assert reads_of_sample({"k_wide_hist": short, "k_wide_reduce": short}, 4096) == 1
    assert reads_of_sample({"k_estimate_one": short}, 256) == 2
