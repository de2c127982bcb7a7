"""Builds libadasd.so (HIP, gfx950 only) and the native half of the binding in-tree with hipcc and g++."""
from __future__ import annotations

import importlib.metadata
import importlib.util
import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libadasd.so")
SOURCES = ["stats.hip", "stats_fused.hip", "decide.hip", "sample.hip", "draft.hip", "shard.hip", "diag.hip", "api.hip"]
HEADERS = [os.path.join(CSRC, h) for h in ("device_common.h", "internal.h", "decide_device.h", "history_device.h",
                                             "sample_device.h", "stats_device.h", "records.h", "noise_series.h")] + [
           os.path.join(os.path.dirname(HERE), "include", "adasd.h")]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         # fused multiply-adds only where the source says fmaf: the same expression must round the
         # same way in every inlined copy (a recomputed partial result has to be bit-identical)
         "-ffp-contract=off",
         # packed-FP32 instructions are kept out of every kernel of this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


NATIVE = os.path.join(HERE, "_native.so")
NATIVE_SRC = os.path.join(CSRC, "py_native.cpp")
NATIVE_FOR = os.path.join(BUILD, "native_for.txt")     # what the extension was built against


def _native_abi() -> str:
    """The extension is tied to the C++ interface of the installed torch and to the interpreter's."""
    return f"torch {importlib.metadata.version('torch')} {sysconfig.get_config_var('SOABI')}"


def _compile_native() -> str:
    """The Python extension, against the headers and libraries of the installed torch."""
    torch = os.path.dirname(importlib.util.find_spec("torch").origin)
    inc = [os.path.join(torch, "include"), os.path.join(torch, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"], "/opt/rocm/include"]
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           *[a for i in inc for a in ("-isystem", i)], NATIVE_SRC, "-o", NATIVE,
           "-L" + os.path.join(torch, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed on {NATIVE_SRC}:\n{res.stderr}")
    with open(NATIVE_FOR, "w") as f:
        f.write(_native_abi())
    return NATIVE


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = ("packed-fp32-ops", "warning generated", "warnings generated")
    msgs = [l for l in res.stderr.splitlines() if l.strip() and not any(n in l for n in noise)]
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{res.stderr}")
    if msgs:
        print("\n".join(msgs))
    return obj


def up_to_date() -> bool:
    """Both libraries are newer than every source and header, and the extension was built against this torch."""
    deps = [os.path.join(CSRC, f) for f in SOURCES] + HEADERS + [NATIVE_SRC]
    newest = max(map(os.path.getmtime, deps))
    if not all(os.path.exists(f) and os.path.getmtime(f) >= newest for f in (LIB, NATIVE)) or not os.path.exists(NATIVE_FOR):
        return False
    with open(NATIVE_FOR) as f:
        return f.read() == _native_abi()


def build(force: bool = True, jobs: int = 4) -> str:
    """Compile every HIP source and link the shared library.  With force=False the build is
    skipped when what is there is up to date."""
    os.makedirs(BUILD, exist_ok=True)
    if not force and up_to_date():
        return LIB
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        native = ex.submit(_compile_native)
        objs = list(ex.map(_compile, SOURCES))
        native.result()
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")
    return LIB


if __name__ == "__main__":
    print(build())
