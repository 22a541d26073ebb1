"""The library's own device code, disassembled: no buffer store of more than 64 bits has its offset in a scalar register.

Behind such a store the compiler lets the next instruction overwrite the data (it waits only where the scalar offset is a constant).
With two waves on a SIMD a kernel stored that next instruction's result in the last four lanes of each sixteen, in a few of a
thousand values, and with one wave never."""
import glob
import os
import re
import shutil
import subprocess

import pytest

LLVM = "/opt/rocm/llvm/bin/"
_STORE = re.compile(r"buffer_store_(?:dwordx[34]|format_xyzw?|short_d16x[34])\s+v\[\d+:\d+\], (?:v\d+|off|v\[\d+:\d+\]), s\[\d+:\d+\], (\S+)")


def stores_with_a_scalar_offset(code):
    """(wide buffer stores, those with a register for a scalar offset)"""
    seen, bad = 0, []
    for line in code:
        m = _STORE.search(line)
        if m:
            seen += 1
            if re.match(r"(s\d|m0|ttmp|vcc)", m.group(1)):
                bad.append(line.split("//")[0].strip())
    return seen, bad


def test_the_search_finds_the_form():
    code = ["\tbuffer_store_dwordx4 v[0:3], v170, s[28:31], s11 offen  // 000\n", "\tbuffer_store_dwordx4 v[0:3], v170, s[28:31], 0 offen  // 008\n",
            "\tbuffer_store_dwordx2 v[0:1], v170, s[28:31], s11 offen  // 010\n"]
    assert stores_with_a_scalar_offset(code) == (2, ["buffer_store_dwordx4 v[0:3], v170, s[28:31], s11 offen"])


@pytest.mark.skipif(not os.path.exists(LLVM + "llvm-objdump"), reason="needs the toolchain's disassembler")
def test_no_wide_store_with_a_scalar_offset(tmp_path):
    from paper_2011_10680_amd import build
    if build.is_stale():
        build.build()
    shutil.copy(build.LIB, tmp_path / "lib.so")
    subprocess.run([LLVM + "llvm-objdump", "--offloading", "lib.so"], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    seen = 0
    for path in glob.glob(str(tmp_path / "*gfx950*")):
        with open(tmp_path / "code.s", "w") as out:
            subprocess.run([LLVM + "llvm-objdump", "-d", path], check=True, stdout=out)
        with open(tmp_path / "code.s") as code:
            n, bad = stores_with_a_scalar_offset(code)
        assert not bad, bad
        seen += n
    assert seen > 100, seen
