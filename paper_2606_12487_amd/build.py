"""Build libdptq.so (gfx950) in-tree with hipcc, and the native half of the
Python binding (_dptq_torch.so, host code) with g++.

    python -m paper_2606_12487_amd.build          # build, print the path

The library is written next to this file so that it travels with the source
tree.  Every HIP source is compiled with IEEE fp32 semantics (no fast-math, no
contraction) because the kernels reproduce a pinned rounding sequence.
"""

import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(PKG_DIR, "_build")
LIB_PATH = os.path.join(PKG_DIR, "libdptq.so")
BINDING_SOURCE = os.path.join(CSRC, "torch_binding.cpp")
BINDING_PATH = os.path.join(PKG_DIR, "_dptq_torch.so")

SOURCES = ["rotate_quant.hip", "decode_fused.hip", "qgemm_ksplit.hip", "range_quant.hip",
           "qgemm.hip", "qgemm_decode.hip", "qgemm_fp6.hip", "qgemm_fp6_ksplit.hip", "kv_quant.hip", "dptq_api.hip"]
ARCH = "gfx950"

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++20", "-fPIC",
    "-ffp-contract=off", "-fno-fast-math",
    # packed fp32 ALU forms are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _hipcc():
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; a ROCm toolchain is required to build libdptq")
    return exe


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"command failed ({res.returncode}): {' '.join(cmd)}\n{out}")
    if verbose and out.strip():
        print(out, flush=True)


def _binding_cmd(out):
    """The g++ command of the binding module, against torch's headers."""
    torch_dir = list(importlib.util.find_spec("torch").submodule_search_locations)[0]
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
            f"-I{torch_dir}/include", f"-I{torch_dir}/include/torch/csrc/api/include",
            f"-I{sysconfig.get_paths()['include']}", f"-I{INCLUDE}", BINDING_SOURCE, "-o", out,
            f"-L{torch_dir}/lib", "-ltorch_python", "-ltorch_cpu", "-lc10", f"-L{PKG_DIR}", "-ldptq",
            "-Wl,-rpath,$ORIGIN"]


def build(verbose=False, jobs=8):
    """Compile every source, link libdptq.so and the binding module; returns the
    library path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    hipcc = _hipcc()
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(BUILD_DIR, src.replace(".hip", ".o"))
        cmd = [hipcc, *HIPCC_FLAGS, f"-I{INCLUDE}", f"-I{CSRC}", "-c",
               os.path.join(CSRC, src), "-o", obj]
        objs.append(obj)
        procs.append(cmd)
    # compile in parallel (bounded)
    running = []
    for cmd in procs:
        if verbose:
            print(" ".join(cmd), flush=True)
        running.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE,
                                              stderr=subprocess.STDOUT, text=True)))
        if len(running) >= jobs:
            _wait(running.pop(0), verbose)
    while running:
        _wait(running.pop(0), verbose)
    tmp = LIB_PATH + ".tmp"
    _run([hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp], verbose)
    os.replace(tmp, LIB_PATH)
    tmp = BINDING_PATH + ".tmp"
    _run(_binding_cmd(tmp), verbose)
    os.replace(tmp, BINDING_PATH)
    return LIB_PATH


def _wait(item, verbose):
    cmd, p = item
    out, _ = p.communicate()
    out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode != 0:
        raise RuntimeError(f"command failed ({p.returncode}): {' '.join(cmd)}\n{out}")
    if verbose and out.strip():
        print(out, flush=True)


if __name__ == "__main__":
    path = build(verbose="-v" in sys.argv)
    print(path)
