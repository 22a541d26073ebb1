"""Compile the HIP sources into ``libhawq.so`` for gfx950 (in-tree, with hipcc), and the Python binding's native half."""
import os
import subprocess
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhawq.so")
# CPython module: argument marshalling in C (host code only).  It is compiled against this interpreter's object layouts, and its
# name says so: another interpreter does not find it and the binding stays with ctypes.
FASTCALL = os.path.join(HERE, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))
OBJ_DIR = os.path.join(HERE, "_build")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def _older(target, deps):
    return not os.path.exists(target) or any(os.path.getmtime(d) > os.path.getmtime(target) for d in deps)


def is_stale():
    """Whether the library, or a native module that was built with it, is older than its sources."""
    header = os.path.join(HERE, "..", "include", "hawq.h")
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [header]
    return _older(LIB, deps) or (os.path.exists(FASTCALL) and _older(FASTCALL, [os.path.join(CSRC, "fastcall.cpp"), header]))


def _compile(src):
    obj = os.path.join(OBJ_DIR, os.path.basename(src)[:-4] + ".o")
    r = subprocess.run([HIPCC] + FLAGS + ["-c", src, "-o", obj], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
    return obj


def _compile_fastcall():
    """Returns None, or why there is no native module: without a host compiler or Python's headers the binding does without."""
    for old in (os.path.join(HERE, "_fastcall.so"), FASTCALL):     # (the first: the name of earlier builds, which every interpreter would load)
        if os.path.exists(old):
            os.remove(old)
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-I", sysconfig.get_paths()["include"],
           "-o", FASTCALL, os.path.join(CSRC, "fastcall.cpp")]
    try:
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    except OSError as e:
        return str(e)
    return None if r.returncode == 0 else r.stdout


def build(force=True, jobs=8):
    """Compile every .hip source and link the shared library; compile the native module, or warn that there is none.  Returns the
    library's path."""
    if not force and not is_stale():
        return LIB
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        fast = ex.submit(_compile_fastcall)
        objs = list(ex.map(_compile, sources()))
        missing = fast.result()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    if missing is not None:
        warnings.warn("the native marshalling module was not built, calls go through ctypes:\n" + missing)
    return LIB


if __name__ == "__main__":
    print(build())
