"""Builds libdp_bk.so (the C-ABI library of HIP kernels) in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdp_bk.so")
PYCALL = os.path.join(HERE, "_pycall" + sysconfig.get_config_var("EXT_SUFFIX"))     # the library's calls for this Python
SOURCES = ["dp_api.hip", "noise.hip", "clip.hip", "fp32_kernels.hip", "ghost.hip", "tn_gemm.hip", "grad_gemm.hip", "grad_packed.hip", "ghost_big.hip", "ghost_brief.hip", "bias.hip", "layerwise.hip", "kept.hip", "ghost_sample.hip", "perex_dma.hip", "perex_narrow.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]
# The gradient kernel's epilogue with noise is 16 copies of a large body; beyond the default size
# limit the compiler stops honouring "#pragma unroll", the accumulator indices stay variable
# and the 256 accumulators move to scratch memory.
# Where the packed rows' loop begins in memory moves the narrow tiles by 5 % (24 layers 768 x 16, 512 x 32 tokens: 257 us at a
# multiple of 64 bytes, up to 272 elsewhere).
PER_FILE_FLAGS = {"grad_gemm.hip": ["-mllvm", "-pragma-unroll-threshold=1000000"], "grad_packed.hip": ["-falign-loops=64"]}


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, *PER_FILE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    objs = []
    for src, obj, proc in procs:
        out, _ = proc.communicate()
        # the host pass does not know the gfx-only feature flag and says so: harmless
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if proc.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
        objs.append(obj)
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(link, check=True)
    build_pycall()
    return LIB


def build_pycall() -> None:
    """The calls with native argument conversion.  Without Python's headers or a host compiler there are none, and the
    binding goes through ctypes."""
    cxx, headers = shutil.which(os.environ.get("CXX", "g++")), sysconfig.get_paths()["include"]
    if os.path.exists(PYCALL):
        os.remove(PYCALL)                                # never one of another build beside the library
    if not cxx or not os.path.exists(os.path.join(headers, "Python.h")):
        print(f"{os.path.basename(PYCALL)} not built: no host C++ compiler or no Python.h; the binding uses ctypes", file=sys.stderr)
        return
    subprocess.run([cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-Wall",
                    "-I", os.path.join(ROOT, "include"), "-I", headers,
                    os.path.join(CSRC, "pycall.cpp"), "-o", PYCALL, "-L", HERE, "-l:libdp_bk.so", "-Wl,-rpath,$ORIGIN"],
                   check=True)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
