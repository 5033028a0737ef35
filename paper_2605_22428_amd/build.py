"""Compile the HIP sources under csrc/ into paper_2605_22428_amd/libmw.so for gfx950, and the calls' Python entry beside it."""
from __future__ import annotations

import glob
import os
import shlex
import shutil
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmw.so")
CALLS = os.path.join(HERE, "_mwcall" + sysconfig.get_config_var("EXT_SUFFIX"))      # (other interpreters do not see it)

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the first kernel argument words are in scalar registers when a wave starts (gfx950 preloads
         # them; a kernel's hottest arguments come first): one memory round trip less per short-lived wave
         "-mllvm", "-amdgpu-kernarg-preload-count=16",
         "-Wall", "-Wno-unused-function"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _c_compiler() -> list:
    """$CC, of any number of words; else the system's compiler; else the one that comes with hipcc."""
    given = shlex.split(os.environ.get("CC", ""))
    return given or [shutil.which("gcc") or shutil.which("cc") or os.path.join(os.path.dirname(_hipcc()), "amdclang")]


def _compile_calls(out: str) -> bool:
    """The extension module through which the binding makes the path's calls; the binding gives it the library's addresses.  Without
    Python's headers there is none, and the binding makes them through ctypes."""
    headers = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(headers, "Python.h")):
        print("no Python.h in %s: the calls go through ctypes" % headers)
        return False
    subprocess.run(_c_compiler() + ["-std=gnu11", "-O2", "-Wall", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"),
                                    "-I", headers, os.path.join(CSRC, "mw_py.c"), "-o", out], check=True)
    return True


def build(verbose: bool = False) -> str:
    """Always compiles; returns the path of the shared library.  Both files are replaced once both are compiled; a module of an
    earlier build does not outlive a library that has none."""
    tmp, tmp_calls = (f + ".tmp%d" % os.getpid() for f in (LIB, CALLS))
    try:
        _compile_library(tmp, verbose)
        calls = _compile_calls(tmp_calls)
        os.replace(tmp, LIB)
        if calls:
            os.replace(tmp_calls, CALLS)
        elif os.path.exists(CALLS):
            os.remove(CALLS)
    finally:
        for f in (tmp, tmp_calls):
            if os.path.exists(f):
                os.remove(f)
    return LIB


def _compile_library(out_path: str, verbose: bool) -> None:
    cmd = [_hipcc()] + FLAGS + ["-I", os.path.join(ROOT, "include"), "-I", CSRC] + sources() + ["-o", out_path]
    if verbose:
        print(" ".join(cmd))
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the device-only feature flag and says so once per use: harmless
    noise = "'-packed-fp32-ops' is not a recognized feature for this target"
    out = "\n".join(l for l in proc.stdout.splitlines() if noise not in l)
    if out.strip():
        print(out)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed with status %d" % proc.returncode)


if __name__ == "__main__":
    print(build(verbose=True))
