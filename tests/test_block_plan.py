"""Where the one-launch bottleneck blocks read their input, checked on the host: the same header the kernel is compiled from, built
with the host compiler."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_rows_beside_the_image_are_addressed_inside_the_tensor(tmp_path):
    exe = str(tmp_path / "block_plan_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-o", exe, os.path.join(HERE, "block_plan_check.cpp")])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0 and int(r.stdout) > 200000, r.stdout
