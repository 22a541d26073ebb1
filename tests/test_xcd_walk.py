"""The tiles that the persistent kernels' workgroups walk, checked on the host: the same header the kernels are compiled from,
built with the host compiler."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_every_tile_once_in_order_of_the_xcds(tmp_path):
    exe = str(tmp_path / "xcd_walk_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-o", exe, os.path.join(HERE, "xcd_walk_check.cpp")])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0 and int(r.stdout) > 4000, r.stdout
