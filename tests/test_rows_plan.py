"""The whole-row 3x3 kernel's tiling arithmetic, walked on the host over its whole range: the same header the kernel is
compiled from, built with the host compiler."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_row_division_lds_layout_and_tile_walk(tmp_path):
    exe = str(tmp_path / "rows_plan_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-o", exe, os.path.join(HERE, "rows_plan_check.cpp")])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
    plans, _, grids, _ = r.stdout.split()
    assert int(plans) > 3000 and int(grids) > 900, r.stdout      # (most widths up to some 130, channels up to 4096 / 8192)
