"""The floating-point form of a block's shortcut term: one fused multiply-add of (256 rb + 1) / 2^(rc+8) and 1.5 * 2^23, rounded to the
nearest even, is (r*rb + 2^(rc-1)) >> rc for every unsigned byte, multiplier below 2^16 and shift from 2 on."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_one_rounding_is_the_shifted_sum():
    g = np.random.default_rng(3)
    r = np.arange(256, dtype=np.int64)[:, None]
    for rc in range(2, 32):
        rb = np.unique(np.concatenate([g.integers(0, 65536, 3000), [0, 1, 2, 3, 65535, 65534, 32768, 1 << min(rc - 1, 15), (1 << min(rc, 16)) - 1]]))[None, :].astype(np.int64)
        factor = 256 * rb + 1
        assert np.array_equal(factor.astype(np.float32).astype(np.int64), factor)          # exact in 24 bits
        p, s = r * factor, rc + 8
        low, half = p & ((1 << s) - 1), 1 << (s - 1)
        nearest = (p >> s) + ((low > half) | ((low == half) & ((p >> s) & 1 == 1)))
        want = (r * rb + (1 << (rc - 1))) >> rc
        assert np.array_equal(nearest, want), rc
        assert want.max() <= 1 << 22


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host C++ compiler")
def test_the_kernels_own_term(tmp_path):
    """... and the functions that the kernel and the network's parameters are made with, built with the host compiler."""
    exe = str(tmp_path / "block_shortcut_check")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-o", exe, os.path.join(HERE, "block_shortcut_check.cpp")])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0 and int(r.stdout) > 20000000, r.stdout
