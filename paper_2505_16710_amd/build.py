"""Build the HIP library (libseco_hip.so) for gfx950 and the extension module of the binding, in-tree.

`python -m paper_2505_16710_amd.build`, or `build_library()` and `build_extension()`.
Objects go to `_build/` next to the sources; the shared objects land in the package
directory, where the binding looks for them.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libseco_hip.so")

SOURCES = [
    "seco_api.hip",
    "seco_select.cpp",
    "elementwise.hip",
    "fwd_f32.hip",
    "kernels_f32.hip",
    "fwd_bf16.hip",
    "fwd4_bf16.hip",
    "fwd4_split_bf16.hip",
    "fwd8_shares_bf16.hip",
    "fwd_small_bf16.hip",
    "bwd_dq_bf16.hip",
    "bwd_dq32_bf16.hip",
    "bwd_dkdv_bf16.hip",
    "bwd_dkdv32_bf16.hip",
    "bwd_fused_bf16.hip",
    "decoder.hip",
    "gemm_bf16.hip",
]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -packed-fp32-ops off: the compiler must not form packed fp32 instructions from scalar code.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I", INCLUDE, "-I", CSRC,
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function", "-Wno-inline-asm"]
# Machine scheduler strategy of the compiler, per source file (measured on the benchmark shapes, every strategy
# tried on every matrix-core kernel): the 8-wavefront forward is 3 % faster with the iterative ILP scheduler than with
# memory (LDS) instructions kept in clauses, the 4-wavefront forward, the dQ and the dK/dV kernels, whose order is fixed
# step by step in the source, 1 - 2 % with the plain ILP one (dK/dV with 32x32x16 products 3 - 7 % slower; dQ with those 3 %
# faster with the iterative one); the launch that holds both passes is slower with either.
SCHED = {"fwd4_bf16.hip": "max-ilp", "bwd_dq_bf16.hip": "max-ilp", "bwd_dkdv_bf16.hip": "max-ilp", "bwd_dq32_bf16.hip": "iterative-ilp", "fwd_bf16.hip": "iterative-ilp", "fwd4_split_bf16.hip": "iterative-ilp",
         "fwd8_shares_bf16.hip": "iterative-ilp"}
SCHED_DEFAULT = "max-memory-clause"
# ... and up to half a per cent when the scheduler does not cluster memory operations
PER_FILE = {"fwd4_bf16.hip": ["-mllvm", "-misched-cluster=false"]}


def _compile(src, extra=()):
    obj = os.path.join(CSRC, "_build", os.path.splitext(src)[0] + ".o")
    sched = ["-mllvm", "-amdgpu-sched-strategy=" + SCHED.get(src, SCHED_DEFAULT)]
    cmd = [HIPCC, *FLAGS, *sched, *PER_FILE.get(src, []), *extra, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(ln for ln in r.stderr.splitlines() if noise not in ln)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_library(verbose=True, extra=(), out=None):
    global LIB
    if out:
        LIB = out
    os.makedirs(os.path.join(CSRC, "_build"), exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, extra), SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    if verbose:
        print(f"built {LIB}")
    return LIB


def build_extension(verbose=True):
    """_seco_ext: the native half of the Python binding (host code only, links against torch's libraries)."""
    import sysconfig

    import torch
    troot = os.path.dirname(torch.__file__)
    out = os.path.join(HERE, "_seco_ext" + sysconfig.get_config_var("EXT_SUFFIX"))
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", INCLUDE,
           "-I", CSRC, "-isystem", os.path.join(troot, "include"), "-isystem", os.path.join(troot, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"),
           os.path.join(CSRC, "binding_ext.cpp"), os.path.join(CSRC, "chunk_step_ext.cpp"), "-o", out, "-L", os.path.join(troot, "lib"),
           "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-ldl"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("building the extension failed:\n" + r.stderr[-4000:])
    if verbose:
        print(f"built {out}")
    return out


if __name__ == "__main__":
    # usage: python -m paper_2505_16710_amd.build [-o out.so] [extra hipcc flags, e.g. -DSECO_DKDV_RB=2]
    argv = sys.argv[1:]
    out = None
    if argv[:1] == ["-o"]:
        out, argv = argv[1], argv[2:]
    build_library(extra=tuple(argv), out=out)
    if out is None:
        build_extension()
