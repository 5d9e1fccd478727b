"""Builds libparo.so (hand-written HIP for gfx950, hipcc) and paro_host.so (the Python calls' native half) in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libparo.so")
HOST_LIB = os.path.join(HERE, "paro_host.so")
OBJ_DIR = os.path.join(HERE, "_build")

SOURCES = ["paro_api.hip", "rotate.hip", "w4_layout.hip", "decode.hip", "decode_wide.hip", "gemm.hip", "linear_rows.hip", "linear_ic.hip", "linear_tile.hip", "quantize.hip", "quantize_weight.hip", "ceilings.hip", "fwht.hip", "mxfp4.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # packed fp32 VALU forms are switched off for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-I", CSRC,
]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{out}")
    if out.strip():
        print(out, file=sys.stderr)
    return obj


def _run(cmd, what: str) -> None:
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{what} failed:\n" + r.stdout)


def _compile_host() -> str:
    from torch.utils import cpp_extension
    obj = os.path.join(OBJ_DIR, "host_call.o")
    dirs = [*cpp_extension.include_paths(), "/opt/rocm/include", sysconfig.get_paths()["include"], INCLUDE]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", *(f"-I{d}" for d in dirs),
          "-c", os.path.join(CSRC, "host_call.cpp"), "-o", obj], "g++ on host_call.cpp")
    return obj


def _link_host(obj: str) -> None:
    from torch.utils import cpp_extension
    _run(["g++", "-shared", "-o", HOST_LIB, obj, f"-L{cpp_extension.library_paths()[0]}", "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip",
          f"-L{HERE}", "-lparo", "-Wl,-rpath,$ORIGIN"], "link of paro_host.so")


def build(verbose: bool = False) -> str:
    """Compile every source (always: no staleness guessing) and link libparo.so and paro_host.so."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        host = ex.submit(_compile_host)
        objs = list(ex.map(_compile, srcs))
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], "link of libparo.so")
    _link_host(host.result())
    if verbose:
        print("built", LIB, HOST_LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
