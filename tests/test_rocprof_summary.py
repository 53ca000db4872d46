"""The counter summaries: what the byte counters are scaled by."""
import sqlite3

from paper_1703_09707_amd import rocprof_summary as RS


def _db(path, rows):
    con = sqlite3.connect(path)
    con.execute("create table counters_collection (kernel_name text, counter_name text, value real, grid_size int)")
    con.execute("create table top_kernels (name text, total_calls int, total_duration real, average real, percentage real)")
    con.execute("create table kernels (name text, duration real, grid_x int, grid_y int, grid_z int)")
    con.executemany("insert into counters_collection values (?, ?, ?, ?)", rows)
    con.execute("insert into top_kernels values ('shoot_fp64_kernel', 1, 5e3, 5.0, 100.0)")
    con.execute("insert into kernels values ('shoot_fp64_kernel', 5e3, 64, 1, 1)")
    con.commit()
    con.close()


def test_bytes_are_scaled_by_the_calibration_copies_alone(tmp_path):
    """Three copies of 8 MiB read half by the counter, beside a run's other
    copies: the scale is 2, whatever those are."""
    copies = [4096.0] * 3 + [1.0, 12.0, 700.0, 0.0]
    fetch, write = str(tmp_path / "f.db"), str(tmp_path / "w.db")
    _db(fetch, [("__amd_rocclr_copyBuffer", "FETCH_SIZE", v, 1) for v in copies]
        + [("shoot_fp64_kernel", "FETCH_SIZE", 100.0, 64)])
    _db(write, [("__amd_rocclr_copyBuffer", "WRITE_SIZE", 2 * v, 1) for v in copies]
        + [("shoot_fp64_kernel", "WRITE_SIZE", 300.0, 64)])
    out = str(tmp_path / "out.txt")
    RS.main(["--kernel", "shoot_fp64_kernel", "--stats", fetch, "--fetch", fetch, "--write", write, "--copy-mib", "8",
             "--out", out])
    s = RS.read_summary(out)
    assert float(s["fetch_scale"]) == 2.0 and float(s["write_scale"]) == 1.0
    assert int(s["traffic_bytes_per_launch"]) == 1024 * (2 * 100 + 300)
