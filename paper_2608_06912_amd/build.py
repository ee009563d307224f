"""Build liblapsum.so in-tree with hipcc for gfx950.

    python -m paper_2608_06912_amd.build          # or __graft_entry__.build()

Every HIP source is compiled for gfx950 only, with packed-FP32 instructions
disabled (-target-feature -packed-fp32-ops); the host orchestration is
compiled without floating-point contraction so that the bracket ranks are
evaluated exactly as written.  Objects go to _build/ next to this file and
the library to liblapsum.so beside it; the native autograd node (a torch
extension over liblapsum.so) to _node.so.
"""
from __future__ import annotations

import concurrent.futures as cf
import importlib.util
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liblapsum.so")
NODE = os.path.join(HERE, "_node.so")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")

HIP_SOURCES = ["row_kernels.hip", "stream_kernels.hip", "sort_kernels.hip",
               "solve_kernels.hip", "bracket_kernels.hip", "band_kernels.hip", "bucket_solve.hip",
               "comparator_kernels.hip", "noalloc.hip",
               "long_solve.hip", "short_rows.hip", "hard_mask.hip"]
HOST_SOURCES = ["lapsum_api.cpp"]
NODE_SOURCE = "autograd_node.cpp"

ARCH = "gfx950"
COMMON = ["-O3", "-std=c++17", "-fPIC", f"-I{INCLUDE}", f"-I{CSRC}"]
HIP_FLAGS = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
HOST_FLAGS = ["-x", "c++", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__"]


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build the LapSum library)")


def _compile(args):
    cmd, src = args
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        err = "\n".join(l for l in proc.stderr.splitlines() if "packed-fp32-ops" not in l)
        raise RuntimeError(f"compiling {src} failed:\n{' '.join(cmd)}\n{err}")
    return src


def _node_compile(hipcc: str, rocm_inc: str, obj: str) -> list:
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    incs = [f"-I{p}" for p in include_paths()] + [f"-I{rocm_inc}",
                                                  f"-I{sysconfig.get_paths()['include']}"]
    return [hipcc, "-O2", "-std=c++17", "-fPIC", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
            "-DTORCH_EXTENSION_NAME=_node", "-DTORCH_API_INCLUDE_EXTENSION_H",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}", *incs, "-c",
            os.path.join(CSRC, NODE_SOURCE), "-o", obj]


def build(verbose: bool = False, jobs: int | None = None) -> str:
    """Compile every source and link liblapsum.so; returns the library path."""
    hipcc = _hipcc()
    os.makedirs(BUILD, exist_ok=True)
    work = []
    objs = []
    for src in HIP_SOURCES:
        obj = os.path.join(BUILD, src + ".o")
        objs.append(obj)
        work.append(([hipcc, *COMMON, *HIP_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj], src))
    rocm_inc = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(hipcc))), "include")
    for src in HOST_SOURCES:
        obj = os.path.join(BUILD, src + ".o")
        objs.append(obj)
        work.append(([hipcc, *COMMON, *HOST_FLAGS, f"-I{rocm_inc}", "-c", os.path.join(CSRC, src),
                      "-o", obj], src))
    jobs = jobs or min(len(work), max(1, min(8, os.cpu_count() or 1)))
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        # the node needs torch's headers, the library nothing but HIP: without
        # torch the library alone is built
        node = None
        if importlib.util.find_spec("torch") is not None:
            node_obj = os.path.join(BUILD, NODE_SOURCE + ".o")
            node = ex.submit(lambda: _compile((_node_compile(hipcc, rocm_inc, node_obj), NODE_SOURCE)))
        for src in ex.map(_compile, work):
            if verbose:
                print(f"compiled {src}", flush=True)
        _link_library(hipcc, objs)
        if verbose:
            print(f"built {LIB}", flush=True)
        if node is None:
            print("torch not found: the native autograd node is not built", flush=True)
            return LIB
        node.result()
    _link_node(hipcc, node_obj)
    if verbose:
        print(f"compiled {NODE_SOURCE}\nbuilt {NODE}", flush=True)
    return LIB


def _run(cmd: list) -> None:
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(f"linking failed:\n{' '.join(cmd)}\n{proc.stderr}")


def _link_library(hipcc: str, objs: list) -> None:
    tmp = LIB + ".tmp"
    _run([hipcc, "-shared", f"--offload-arch={ARCH}", "-Wl,-soname,liblapsum.so", "-o", tmp, *objs])
    os.replace(tmp, LIB)


def _link_node(hipcc: str, node_obj: str) -> None:
    import torch
    tlib = os.path.join(os.path.dirname(torch.__file__), "lib")
    tmp = NODE + ".tmp"
    _run([hipcc, "-shared", "-o", tmp, node_obj, LIB, f"-L{tlib}", "-lc10", "-lc10_hip",
          "-ltorch_cpu", "-ltorch_python", "-ltorch", "-Wl,-rpath,$ORIGIN"])
    os.replace(tmp, NODE)


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
