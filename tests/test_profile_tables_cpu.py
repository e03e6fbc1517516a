"""What bench.py reads back from the profile summaries: the dominant kernel's time and its HBM bytes belong together."""
import csv

import pytest

TRACE = ("| Kernel | Grid (threads) | Calls | Median | Average | Min | Max |\n|---|---|---|---|---|---|---|\n"
         "| `page_score_long_kernel<4, true, 4>` | 2048x64x4 | 205 | 61151 | 61519 | 60111 | 67391 |\n")
TRAFFIC = ("| Kernel | Grid (threads) | Dispatches | FETCH_SIZE KiB | WRITE_SIZE KiB | HBM bytes per dispatch (scaled) |\n"
           "|---|---|---|---|---|---|\n| `%s` | %d | 42 | 33122 | 2120 | 69994438 |\n")


@pytest.mark.parametrize("name,threads,traffic", [
    ("page_score_long_kernel<4, true, 4>", 2048 * 64 * 4, 69994438),
    ("page_score_long_kernel<4, true, 4>", 2048 * 64, None),            # another launch of that kernel
    ("page_score_kernel<4, true, 4>", 2048 * 64 * 4, None)])            # another kernel of the stage
def test_traffic_is_that_of_the_traced_kernel(tmp_path, monkeypatch, name, threads, traffic):
    import bench
    monkeypatch.setattr(bench, "PROFILES", str(tmp_path))
    (tmp_path / "c2_decode_step_kernel_trace.md").write_text(TRACE)
    (tmp_path / "c2_decode_step_hbm_traffic.md").write_text(TRAFFIC % (name, threads))
    got = bench.profile_figures("page_score")
    assert got["rocprofv3_kernel_us"] == pytest.approx(61.519)
    assert got["traffic"] == traffic and (got["traffic_source"] is None) == (traffic is None)


def test_a_trace_names_all_three_dimensions_of_the_grid(tmp_path):
    from paper_2502_02770_amd.rocprof_summary import read_trace_table, write_trace
    row = {"Kernel_Name": "void (anonymous namespace)::page_score_kernel<4, true, 4>(ScoreArgs)", "Start_Timestamp": 100,
           "End_Timestamp": 1100, "Grid_Size_X": 2048, "Grid_Size_Y": 64, "Grid_Size_Z": 8}
    with open(tmp_path / "t_kernel_trace.csv", "w", newline="") as f:
        w = csv.DictWriter(f, list(row))
        w.writeheader()
        w.writerow(row)
    with open(tmp_path / "t.md", "w") as f:
        write_trace(str(tmp_path), "title", "command", f)
    assert read_trace_table(str(tmp_path / "t.md")) == {
        "page_score_kernel<4, true, 4>": {"threads": 2048 * 64 * 8, "calls": 1, "median_ns": 1000, "avg_ns": 1000}}
