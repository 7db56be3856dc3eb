"""The kernel summary's launch table follows the order in which the launches ran, whatever
order the trace lists them in."""
import csv
import json

from paper_2312_04356_amd import prof_summary


def test_launch_table_is_in_time_order(tmp_path, capsys):
    names = ["void nj::k_ntt_tile_gal(int)", "void nj::k_bconv_col<16>(int)", "void nj::k_ntt_ip<3, true, true>(int)",
             "void nj::k_moddown_multi(int)"]
    rows = [{"Kernel_Name": n, "Start_Timestamp": 1000 * i, "End_Timestamp": 1000 * i + 500, "Workgroup_Size_X": 256,
             "Grid_Size_X": 512, "Grid_Size_Y": 1, "Grid_Size_Z": 1, "VGPR_Count": 32, "LDS_Block_Size": 0}
            for i, n in enumerate(["void nj::k_zero(int)"] + names)]
    trace = tmp_path / "trace.csv"
    with open(trace, "w", newline="") as f:
        w = csv.DictWriter(f, rows[0].keys())
        w.writeheader()
        w.writerows(rows[i] for i in (4, 0, 2, 3, 1))
    kernels = {k: {"launches_per_step": 1, "ms_per_step": 0.1, "avg_launch_us": 100.0}
               for k in ("k_ntt_tile<true>", "k_bconv", "k_key_ip", "other")}
    bench = {"config": {"workload": "w"}, "steps": 1, "value": 1.0, "pipeline": {"kernels": kernels},
             "roofline": {"kernel": "k_key_ip", "avg_launch_us": 1.0, "achieved": 1.0, "frac": 0.1}}
    js = tmp_path / "bench.json"
    js.write_text(json.dumps(bench) + "\n")
    prof_summary.main(str(trace), str(js), str(js), "cmd")
    table = capsys.readouterr().out.split("launch by launch")[1]
    got = [line.split("|")[2].strip() for line in table.splitlines() if line.startswith("| ") and line[2].isdigit()]
    assert got == ["k_ntt_tile_gal", "k_bconv_col<16>", "k_ntt_ip<3, true, true>", "k_moddown_multi"]
