"""Builds in-tree: libnd.so (HIP, gfx950) with hipcc, no torch involved; _nd_call.so (the Python side's marshalling of
tensors, csrc/nd_python.cpp) with a host compiler against torch's headers, where there is a torch: callers of the C ABI
need only the first."""
from __future__ import annotations

import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libnd.so")
CALL_LIB = os.path.join(HERE, "_nd_call.so")
SOURCES = ["nd_api.hip", "nd_graph.hip", "nd_sort.hip", "nd_sched.hip", "nd_sample.hip", "nd_khop.hip", "nd_walk.hip", "nd_walk_free.hip", "nd_layer.hip", "nd_edges.hip", "nd_pack.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if warn:
        sys.stderr.write(warn + "\n")
    return obj


def _host_compiler() -> str:
    """g++, or the clang++ that hipcc itself uses for host code."""
    return os.environ.get("CXX") or shutil.which("g++") or os.path.join(os.path.dirname(HIPCC), "amdclang++")


def _compile_marshalling() -> None:
    if importlib.util.find_spec("torch") is None:
        sys.stderr.write("torch is not installed: libnd.so is built without the Python binding's _nd_call.so\n")
        return
    import torch
    root = os.path.dirname(torch.__file__)
    cmd = [_host_compiler(), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], os.path.join(CSRC, "nd_python.cpp"), "-o", CALL_LIB,
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"the host compiler failed for nd_python.cpp:\n{r.stdout}\n{r.stderr}")


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=6) as ex:
        marshalling = ex.submit(_compile_marshalling)
        objs = list(ex.map(_compile, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    marshalling.result()  # after the link: libnd.so does not depend on it
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
