"""Build the HIP library in-tree:  python -m paper_2301_10936_amd.build

hipcc cross-compiles for gfx950 without a GPU.  The result, libpit_hip.so, sits next to this file
and is what the binding loads; _pit_native.so beside it is the native part of that binding.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpit_hip.so")
SOURCES = ["pit_api.hip", "pit_index.hip", "pit_gemm.hip", "pit_gemm_m.hip", "pit_gemm_ring.hip", "pit_gemm_m_ring.hip", "pit_slab.hip", "pit_moe.hip", "pit_attn.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wno-inline-asm", "-Wno-pass-failed",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# Options of one source, left out where the compiler does not know them.
# -amdgpu-mfma-vgpr-form: matrix results in vector registers.  The 128-row k_slab_strip_tall adds them to values from LDS and
# pays a register move per element otherwise (4096^3, 1 x 32 micro-tiles, 10 % kept: 157 us with, 163 without; 1 x 64 at
# 50 % 269, 282).  No other kernel gains, and the hand-placed distances between matrix instructions in pit_gemm.hip are
# those of code generated without it.
OPTIONAL = {"pit_slab.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"]}


BINDING = os.path.join(HERE, "_pit_native.so")        # pit.py's way into the library for the calls of every step (host code)
PROBE_LIB = os.path.join(HERE, "libpit_probe.so")     # measurement probes (bench_micro.py --probe), not the product


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    noise = "is not a recognized feature for this target"
    return proc.returncode, "\n".join(l for l in proc.stdout.splitlines() if noise not in l)


def _compile(src, obj, verbose):
    optional = OPTIONAL.get(os.path.basename(src), [])
    rc, out = _run(["hipcc", *FLAGS, *optional, "-c", "-o", obj, src], verbose)
    if rc != 0 and optional and "unknown command line argument" in out.lower():
        rc, out = _run(["hipcc", *FLAGS, "-c", "-o", obj, src], verbose)
    if rc != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out, flush=True)


def _library(srcs, lib, verbose):
    with tempfile.TemporaryDirectory() as tmp, concurrent.futures.ThreadPoolExecutor(4) as pool:
        objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in srcs]
        list(pool.map(_compile, srcs, objs, [verbose] * len(srcs)))
        rc, out = _run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib, *objs], verbose)
    if rc != 0:
        raise RuntimeError("hipcc failed:\n" + out)


def _binding(lib, verbose):
    import sysconfig
    import torch
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    rc, out = _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                    "-I" + sysconfig.get_paths()["include"], "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"),
                    os.path.join(CSRC, "pit_binding.cpp"), "-o", BINDING, "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"),
                    "-ltorch_python", "-ltorch_cpu", "-lc10", "-L" + HERE, "-l:" + os.path.basename(lib), "-Wl,-rpath,$ORIGIN"], verbose)
    if rc != 0:
        raise RuntimeError("building the binding failed:\n" + out)


def build(verbose: bool = False) -> str:
    srcs = [os.path.join(CSRC, s) for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    _library(srcs, LIB, verbose)
    _binding(LIB, verbose)
    _library([os.path.join(CSRC, "pit_probe.hip")], PROBE_LIB, verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
