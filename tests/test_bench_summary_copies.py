"""bench.py's counter summary calibrates on the runtime's 1 GiB device copy, not
on a kernel of the library that has "copy" in its name (state_copy_kernel, whose
grid is the larger)."""
import csv

import bench


def test_calibration_ignores_the_librarys_copies(tmp_path, capsys):
    hdr = ["Dispatch_Id", "Kernel_Name", "Grid_Size", "Counter_Name", "Counter_Value",
           "Start_Timestamp", "End_Timestamp"]
    rows = [[4, "__amd_rocclr_copyBuffer", 131072, "FETCH_SIZE", 524288, 0, 400_000],
            [7, "void nb::(anonymous namespace)::state_copy_kernel<false>(x)", 41943040, "FETCH_SIZE", 360462,
             400_000, 500_000],
            [9, "void nb::(anonymous namespace)::force_kernel<0, 1, 4, false, false>(x)", 1048576,
             "FETCH_SIZE", 1000, 500_000, 7_000_000]]
    with open(tmp_path / "f_counter_collection.csv", "w", newline="") as f:
        csv.writer(f).writerows([hdr, *rows])
    bench.summarize_profile(str(tmp_path))
    out = capsys.readouterr().out
    assert "factor 2.0000" in out and "-> 2.05 MB per launch" in out
    assert "state_copy" not in out
