"""Builds libdastac_hip.so (all HIP sources under csrc/, gfx950 only) with hipcc."""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdastac_hip.so")
# The binding's native calls: host code for this interpreter and no other, hence its tag in the name.  Without the interpreter's headers
# the binding goes through ctypes.
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))

# Packed-fp32 VALU forms are switched off for the device pass (the host pass warns that it does
# not know the feature; harmless).
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
    subprocess.check_call(["hipcc", *HIPCC_FLAGS, "-c", src, "-o", obj])
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, sources()))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    for old in glob.glob(os.path.join(HERE, "_calls*.so")):
        os.remove(old)
    include = sysconfig.get_paths()["include"]
    if os.path.exists(os.path.join(include, "Python.h")):
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-Wno-missing-field-initializers",
                               "-I", include, os.path.join(CSRC, "calls.cpp"), "-o", CALLS])
    else:
        print("no Python.h in %s: calls go through ctypes" % include)
    return LIB


if __name__ == "__main__":
    print(build())
