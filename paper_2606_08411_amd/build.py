"""Build the HIP library libasynclane.so in-tree for gfx950.

Each source is compiled to an object in ``_build/`` with hipcc (in parallel),
then linked into ``paper_2606_08411_amd/libasynclane.so``; the CPython module
``_fast.so`` is one more command.  Runs on a machine
without a GPU (hipcc cross-compiles).
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libasynclane.so")
FAST = os.path.join(PKG, "_fast.so")   # CPython module (csrc/fast_call.cpp)
SOURCES = (["abi.cpp", "scheduler.cpp", "lane_attn.hip", "lmhead.hip", "select_unmask.hip"] +
           [f"lmhead_tile_{g}.hip" for g in "abcdefghij"])
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         # keep the compiler away from packed-fp32 instructions
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-Wall", "-Wno-unused-function"]


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass warns that it does not know the packed-fp32 feature
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"command failed: {' '.join(cmd)}\n{err}")
    return err


def _fast_command(out):
    """Host compiler command of the CPython module (no device code)."""
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    inc = [x for p in include_paths() + [sysconfig.get_paths()["include"]] for x in ("-isystem", p)]
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + inc +
            [os.path.join(CSRC, "fast_call.cpp"), "-o", out, "-L" + lib, "-lc10", "-ltorch_cpu",
             "-ltorch_python"])


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    objs = []
    cmds = []
    for s in SOURCES:
        obj = os.path.join(BUILD, os.path.splitext(s)[0] + ".o")
        objs.append(obj)
        cmds.append([HIPCC, "-x", "hip", "-c", os.path.join(CSRC, s), "-o", obj] + FLAGS)
    with ThreadPoolExecutor(8) as ex:
        fast = ex.submit(lambda: _run(_fast_command(FAST + ".tmp")))
        for err in ex.map(_run, cmds):
            if verbose and err.strip():
                print(err, file=sys.stderr)
    tmp = LIB + ".tmp"
    _run([HIPCC, "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    fast.result()   # (the library is usable without the module)
    os.replace(FAST + ".tmp", FAST)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
