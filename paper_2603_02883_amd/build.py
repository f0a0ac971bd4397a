"""Builds libfb4.so (the C-ABI library with its gfx950 kernels; hipcc) and _fb4call (the Python binding's calls into it; the host
compiler) in-tree.  The library serves every Python; the module is one interpreter's, named after it, and is left out where that
interpreter's headers or a host compiler are missing: the binding then makes its calls through ctypes."""

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfb4.so")
CALL = os.path.join(HERE, "_fb4call" + sysconfig.get_config_var("EXT_SUFFIX"))
CALL_SOURCE = os.path.join(CSRC, "fb4_pycall.c")
OBJ_DIR = os.path.join(HERE, "_build")
# one translation unit per group of entry points, compiled side by side
SOURCES = [os.path.join(CSRC, f) for f in ("fb4_api.hip", "fb4_producers.hip", "fb4_attention.hip")]
HEADER = os.path.join(os.path.dirname(HERE), "include", "fb4.h")
DEPS = SOURCES + [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith(".hpp")] + [HEADER]
PYTHON_INCLUDE = sysconfig.get_paths()["include"]
HOST_CC = os.environ.get("CC", "gcc")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 instructions stay off for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the dispatcher fills up to 16 leading kernel-argument registers before a wavefront starts
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-function",
]
# the host pass does not know the device-only feature flag and says so
NOISE = "is not a recognized feature for this target"


def _newer(target, sources):
    return os.path.exists(target) and all(os.path.getmtime(d) <= os.path.getmtime(target) for d in sources)


def can_build_call():
    """Whether this interpreter's headers and a host compiler are here."""
    return os.path.exists(os.path.join(PYTHON_INCLUDE, "Python.h")) and shutil.which(HOST_CC.split()[0]) is not None


def up_to_date():
    return _newer(LIB, DEPS) and (_newer(CALL, [CALL_SOURCE, HEADER]) or not can_build_call())


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if NOISE not in l)
    if r.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (cmd[0], err))
    return err


def build_call():
    """Compile the binding's C module for this interpreter against the library that is there."""
    new = "%s.%d" % (CALL, os.getpid())   # (another process may be loading, or building, the same one)
    try:
        err = _run(HOST_CC.split() + ["-O2", "-Wall", "-shared", "-fPIC", "-I" + PYTHON_INCLUDE, "-o", new, CALL_SOURCE, "-L" + HERE,
                                      "-l:" + os.path.basename(LIB), "-Wl,-rpath,$ORIGIN"])
        os.replace(new, CALL)
    finally:
        if os.path.exists(new):
            os.remove(new)
    return err


def build(force=True, verbose=False):
    """Compile the library and the module.  force=False skips the compile when both are newer than their sources."""
    if not force and up_to_date():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ_DIR, exist_ok=True)
    objs = [os.path.join(OBJ_DIR, os.path.basename(s)[:-4] + ".o") for s in SOURCES]
    with ThreadPoolExecutor(max_workers=len(SOURCES)) as pool:
        errs = list(pool.map(lambda so: _run([hipcc] + HIPCC_FLAGS + ["-c", so[0], "-o", so[1]]), zip(SOURCES, objs)))
    errs.append(_run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs))
    if can_build_call():
        errs.append(build_call())
    if verbose and any(e.strip() for e in errs):
        print("\n".join(e for e in errs if e.strip()), file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
