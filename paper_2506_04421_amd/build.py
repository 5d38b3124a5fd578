"""Builds libhmar_attn.so (HIP kernels + C ABI, hipcc for gfx950) and _launch.so (the binding's native call
path, host code only) in-tree."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libhmar_attn.so")
LAUNCH_PATH = os.path.join(HERE, "_launch.so")

SOURCES = ["api.cpp", "schedule.cpp", "fwd.hip", "bwd.hip", "no_alloc.hip"]

# -packed-fp32-ops off: hipcc must not form v_pk_*_f32 from the fp32 softmax arithmetic.
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc_path() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def variant_path(name: str) -> str:
    """Where a measurement variant of the library is written (never the library the package loads)."""
    return os.path.join(HERE, f"libhmar_attn_{name}.so")


def launch_command(out: str, defines=()) -> list:
    """g++ command of the Python module _launch: host code against torch's C++ interface, no device code."""
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc_path())))
    return [shutil.which("g++") or "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", os.path.join(ROOT, "include"),
            "-I", inc, "-I", os.path.join(inc, "torch", "csrc", "api", "include"), "-I", os.path.join(rocm, "include"),
            "-I", sysconfig.get_paths()["include"], *[f"-D{d}" for d in defines], os.path.join(CSRC, "py_launch.cpp"),
            "-L", lib, "-lc10", "-ltorch_cpu", "-ltorch_python", "-lc10_hip", "-ltorch_hip", "-o", out]


def build_library(verbose: bool = False, variant: str = "", defines=()) -> str:
    """Compile every source: the shared library and, beside it, the binding's _launch module.  Always
    recompiles.  With `variant`, builds libhmar_attn_<variant>.so alone with the given -D knobs (see the
    list at the top of csrc/device_common.h) next to the library instead: for measurements only."""
    out = variant_path(variant) if variant else LIB_PATH
    jobs = [(out, [hipcc_path(), "-O3", "-std=c++17", "-fPIC", "-shared", "-x", "hip", *DEVICE_FLAGS,
                   "-I", os.path.join(ROOT, "include"), "-I", CSRC, *[f"-D{d}" for d in defines],
                   *[os.path.join(CSRC, s) for s in SOURCES], "-o", out + ".tmp"])]
    if not variant:
        jobs.append((LAUNCH_PATH, launch_command(LAUNCH_PATH + ".tmp")))
    procs = []
    for target, cmd in jobs:
        if verbose:
            print(" ".join(cmd), flush=True)
        try:
            procs.append((target, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        except OSError as e:                        # no such compiler
            procs.append((target, e))
    results = [(target, *((str(proc) + "\n", 1) if isinstance(proc, OSError) else (proc.communicate()[0], proc.returncode)))
               for target, proc in procs]
    for target, _, code in results:                 # the library is of use without the module
        if code == 0:
            os.replace(target + ".tmp", target)
    for target, log, code in results:
        if code != 0:
            sys.stderr.write(log)
            raise RuntimeError(f"the compiler failed building {os.path.basename(target)}")
    return out


if __name__ == "__main__":
    import argparse
    ap = argparse.ArgumentParser(description=__doc__)
    ap.add_argument("--variant", default="", help="build libhmar_attn_<variant>.so for measurements")
    ap.add_argument("-D", dest="defines", action="append", default=[], help="macro for the variant, e.g. -DHMAR_TUNE_LDS_PAD_FWD=32768")
    a = ap.parse_args()
    if a.defines and not a.variant:
        ap.error("-D knobs need --variant: the library the package loads is always built without them")
    print(build_library(verbose=True, variant=a.variant, defines=a.defines))
