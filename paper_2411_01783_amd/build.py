"""Build libcp_attn.so (HIP, gfx950 only, with hipcc) and the CPython module _py_calls.so of
binding.py (host C++, with g++) in-tree.

Usage: python -m paper_2411_01783_amd.build [--force]
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJ_DIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libcp_attn.so")
PY_SRC = os.path.join(CSRC, "py_calls.cpp")
PY_LIB = os.path.join(HERE, "_py_calls.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",  # no packed-fp32 codegen
    "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
    "-I", INCLUDE, "-I", CSRC,
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _newest_dep() -> float:
    deps = sources() + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(INCLUDE, "*.h"))
    return max(os.path.getmtime(p) for p in deps)


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.basename(src) + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines()
                    if "is not a recognized feature for this target" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_py_calls(force: bool = False) -> str:
    """Compile _py_calls.so against this interpreter's and torch's headers. Returns its path."""
    header = os.path.join(INCLUDE, "cp_attn.h")
    if not force and os.path.exists(PY_LIB) and \
            os.path.getmtime(PY_LIB) >= max(os.path.getmtime(p) for p in (PY_SRC, header)):
        return PY_LIB
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    tmp = PY_LIB + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I", INCLUDE, "-isystem", os.path.join(root, "include"),
           "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-I", sysconfig.get_paths()["include"], PY_SRC, "-o", tmp,
           "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed for %s:\n%s" % (PY_SRC, res.stderr))
    if res.stderr.strip():
        sys.stderr.write(res.stderr)
    os.replace(tmp, PY_LIB)
    return PY_LIB


def build(force: bool = False, jobs: int = 4) -> str:
    """Compile every csrc/*.hip for gfx950 and link libcp_attn.so, and the module of the
    binding's calls. Returns the library's path."""
    build_py_calls(force)
    if not force and os.path.exists(LIB) and os.path.getmtime(LIB) >= _newest_dep():
        return LIB
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, sources()))
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
