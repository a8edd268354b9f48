"""Build the gfx950 library in-tree: hipcc -> paper_2306_14316_amd/libim2win.so, and, for the interpreter that runs this, gcc -> the module _native."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libim2win.so")
NATIVE = os.path.join(HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))
OBJDIR = os.path.join(HERE, "_build")
SOURCES = ("api.hip", "transform.hip", "conv_basic.hip", "conv_mfma.hip", "conv_mfma_fast.hip", "conv_split.hip",
           "conv_split_stem.hip", "conv_split_1x1.hip", "conv_mfma_shallow.hip", "conv_mfma_1x1.hip", "baselines.hip", "probes.hip")
# Packed-fp32 VALU instructions are switched off for all device code.
DEVICE_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
                "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *DEVICE_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stderr))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _build_native() -> None:
    """The binding's short path (host code, a CPython module).  Without gcc or Python's headers there is none, and the binding does without."""
    tmp = NATIVE + ".tmp.%d" % os.getpid()
    try:
        subprocess.run(["gcc", "-O2", "-Wall", "-shared", "-fPIC", "-I" + sysconfig.get_paths()["include"],
                        os.path.join(CSRC, "native_call.c"), "-o", tmp], check=True)
        os.replace(tmp, NATIVE)
    except (OSError, subprocess.CalledProcessError) as e:
        if os.path.exists(NATIVE):   # (of an earlier build, perhaps of other sources)
            os.remove(NATIVE)
        sys.stderr.write("warning: the module _native was not built (%s); calls take the general path, some 2 us slower\n" % e)


def build(verbose: bool = False) -> str:
    """Compile every source for gfx950 and link the shared library (always rebuilds); the binding's module with it."""
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    _build_native()
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
