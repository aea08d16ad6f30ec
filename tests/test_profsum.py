"""The profile summaries find a compress call's EM dispatches, of the built-in
launches (batches planned in one launch, without k_plan_reset) and of one launch
per bucket."""
import csv
import os

import numpy as np
import pytest

from paper_2007_12273_amd import _lib, profsum

BUILT_IN = ["void gm::k_moments<3>(gm::CompressArgs)", "void gm::k_plan_scan<3>(gm::CompressArgs, int)",
            "void gm::k_em<3, 16, 8, false, float, true>(gm::CompressArgs)",
            "void gm::k_em_span<3, 16, 8, float, 1, 8>(gm::CompressArgs, int, int, int)",
            "void gm::k_em_span<3, 16, 8, float, 1, 8>(gm::CompressArgs, int, int, int)",
            "void gm::k_em_big<3, 16, float>(gm::CompressArgs)", "void gm::k_finish<3, 16, true>(gm::CompressArgs)"]
PER_BUCKET = ["void gm::k_moments<3>(gm::CompressArgs)", "gm::k_plan_reset(int*)",
              "void gm::k_em<3, 16, 2, true, float, false>(gm::CompressArgs)",
              "void gm::k_em<3, 16, 4, true, float, false>(gm::CompressArgs)",
              "void gm::k_finish<3, 16, true>(gm::CompressArgs)"]


def _write(path, extra):
    """One call of each form; a dispatch lasts 1 ms and starts 1 ms after the last."""
    rows = [dict(Kernel_Name=n, Dispatch_Id=i + 1, Start_Timestamp=1000000 * i, End_Timestamp=1000000 * (i + 1),
                 Queue_Id=1 + i % 4, Workgroup_Size=1024 if "true>" in n else 64, **extra)
            for i, n in enumerate(BUILT_IN + PER_BUCKET)]
    with open(path, "w") as f:
        w = csv.DictWriter(f, rows[0].keys())
        w.writeheader()
        w.writerows(rows)
    return str(path)


def test_trace_of_both_forms(tmp_path, capsys):
    profsum.main(["trace", _write(tmp_path / "t.csv", {})])
    out = capsys.readouterr().out
    assert "k_em<3,16,8,false,float,true>+0.001.00q3" in out.replace(" ", "")
    assert "call  0:  4 EM dispatches, span    4.000 ms" in out and "call  1:  2 EM dispatches, span    2.000 ms" in out


def test_bytes_of_both_forms(tmp_path, capsys):
    f = _write(tmp_path / "f.csv", dict(Counter_Name="FETCH_SIZE", Counter_Value=10))
    w = _write(tmp_path / "w.csv", dict(Counter_Name="WRITE_SIZE", Counter_Value=3))
    profsum.main(["bytes", f, w])
    out = capsys.readouterr().out.split("\n")
    assert out[2].split()[-3::2] == ["40", "12"] and out[3].split()[-3::2] == ["20", "6"], out


def test_instructions_per_wave_update(tmp_path, capsys):
    """Cells of 100, 1500 and 3000 particles run one, four and eight waves."""
    if not os.path.exists(_lib.LIB_PATH):
        pytest.skip("library not built")
    c = _write(tmp_path / "c.csv", dict(Counter_Name="SQ_INSTS_VALU", Counter_Value=52.5))
    np.savez(tmp_path / "v.npz", n=np.array([100, 1500, 3000]), visits_cold=np.array([2, 1, 1]))
    profsum.main(["insts", str(tmp_path / "v.npz"), "0:cold", c])
    out = capsys.readouterr().out
    assert "4 component updates, 14 wave-updates" in out and "15.00 per wave-update" in out, out
