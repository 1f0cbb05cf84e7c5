"""Compiles the HIP sources in csrc/ into libomnistep.so (gfx950) and the host-call extension in pyext/, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libomnistep.so")
EXT = os.path.join(HERE, "_hostcall" + sysconfig.get_config_var("EXT_SUFFIX"))

# Packed-fp32 VALU forms are switched off for every device compile.
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes"]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def build(verbose: bool = False, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

    def compile_one(src):
        obj = os.path.join(OBJ, src + ".o")
        cmd = [hipcc, *COMMON, "-c", os.path.join(CSRC, src), "-o", obj]
        if src.endswith(".hip"):
            cmd[1:1] = DEVICE_FLAGS
        else:
            # host code: no fused multiply-adds (the measured-time controller's doubles must repeat bit for bit)
            cmd[1:1] = ["-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-ffp-contract=off"]
            cmd[0] = os.environ.get("CXX", "g++")
        r = subprocess.run(cmd, capture_output=True, text=True)
        if verbose or r.returncode != 0:
            sys.stderr.write(" ".join(cmd) + "\n" + r.stdout + r.stderr)
        if r.returncode != 0:
            raise RuntimeError(f"compiling {src} failed")
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, sources()))
    cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(" ".join(cmd) + "\n" + r.stdout + r.stderr)
        raise RuntimeError("linking libomnistep.so failed")
    for f in os.listdir(HERE):                       # of another interpreter, or without its tag
        if f.startswith("_hostcall.") and f.endswith(".so"):
            os.remove(os.path.join(HERE, f))
    include = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(include, "Python.h")):
        sys.stderr.write(f"no Python.h under {include}: the calls of every step marshal their arguments through ctypes\n")
        return LIB
    cmd = [os.environ.get("CXX", "g++"), *COMMON, "-shared", "-I" + include,
           os.path.join(HERE, "pyext", "hostcall.cpp"), "-o", EXT]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(" ".join(cmd) + "\n" + r.stdout + r.stderr)
        raise RuntimeError("compiling hostcall.cpp failed")
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
