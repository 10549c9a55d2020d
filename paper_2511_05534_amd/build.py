"""Builds libflowmm.so (gfx950) from csrc/*.hip with hipcc, and the CPython module that calls it, in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libflowmm.so")
CALLS = os.path.join(HERE, "_flowmm_calls.so")
SOURCES = ["flowmm_api.hip", "profile.hip", "meta.hip", "score.hip", "select.hip", "match.hip", "select_match.hip", "merge.hip", "unit_path.hip", "flow_exact.hip", "decode.hip", "cache.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src.replace(".hip", ".o"))
    cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_library(jobs: int = 6) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + f".tmp{os.getpid()}"
    subprocess.check_call([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    _build_calls()
    return LIB


def _build_calls():
    """The extension module finds the library beside itself."""
    tmp = CALLS + f".tmp{os.getpid()}"
    subprocess.check_call([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
                           "-I" + sysconfig.get_paths()["include"], os.path.join(CSRC, "python_calls.cpp"),
                           "-L" + HERE, "-lflowmm", "-Wl,-rpath,$ORIGIN", "-o", tmp])
    os.replace(tmp, CALLS)


def library_path() -> str:
    return LIB


def calls_path() -> str:
    return CALLS


if __name__ == "__main__":
    print(build_library())
