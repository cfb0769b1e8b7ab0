"""Builds libhdt.so (HIP kernels + C ABI) for gfx950 with hipcc, and the Python module of its hot calls, in-tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig

_PKG = os.path.dirname(os.path.abspath(__file__))
_ROOT = os.path.dirname(_PKG)
CSRC = os.path.join(_PKG, "csrc")
LIB = os.path.join(_PKG, "libhdt.so")
# compiled for one Python (the suffix says which) and one torch; libhdt.so takes any of both
PYCALL = os.path.join(_PKG, "_hdt_pycall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
SOURCES = ["hdt_api.hip", "hdt_layout.hip", "hdt_f32.hip", "hdt_fwd.hip", "hdt_bwd.hip", "hdt_hpe.hip", "hdt_cross.hip", "hdt_probe.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    # no packed fp32 instructions: some of their forms have given wrong results on this hardware
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no NaN-quieting v_max(x, x) in front of every fmaxf: wherever a NaN can stand (rows of pad positions may
    # hold anything) it is removed by a select before any arithmetic looks at it, and the kernels produce none
    # on their own (infinities are still honoured)
    "-fno-honor-nans",
    "-Wno-unused-command-line-argument",
    # the direct-to-LDS loads set M0 inside their asm block and list it as clobbered
    "-Wno-inline-asm",
]


def _pycall_command():
    """The host compiler's line for the Python module (against torch's headers; no device code)."""
    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DHDT_TORCH_VERSION="{torch.__version__}"',
            "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include/torch/csrc/api/include"),
            "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
            "-I", os.path.join(_ROOT, "include"), os.path.join(CSRC, "hdt_pycall.cpp"), "-o", PYCALL,
            "-L", os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10_hip", "-lc10"]


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared library and the Python module.  Always recompiles.  The module needs g++ and the
    headers of torch and Python; where it cannot be made the library is linked all the same, and this raises behind that."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        cmd = [hipcc, *HIPCC_FLAGS, "-I", os.path.join(_ROOT, "include"), "-I", CSRC, "-c",
               os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = []
    for old in glob.glob(os.path.join(os.path.dirname(PYCALL), "_hdt_pycall*.so")):
        os.remove(old)  # made for the library of an earlier build
    module = "hdt_pycall.cpp"
    try:
        cmd = _pycall_command()
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((module, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    except (ImportError, OSError) as e:  # no torch, no compiler
        failed.append(module)
        print(f"[build] {module} FAILED\n{e}", file=sys.stderr)
    for src, p in procs:
        log, _ = p.communicate()
        log = "\n".join(l for l in log.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            failed.append(src)
            print(f"[build] {src} FAILED\n{log}", file=sys.stderr)
        elif verbose and log.strip():
            print(log)
    if any(src != module for src in failed):
        raise RuntimeError("hipcc failed")
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    if failed:
        raise RuntimeError(f"{LIB} is built, the Python module of its hot calls (_hdt_pycall) is not")
    return LIB


if __name__ == "__main__":
    import argparse
    ap = argparse.ArgumentParser()
    ap.add_argument("-v", "--verbose", action="store_true")
    a = ap.parse_args()
    print(build(verbose=a.verbose))
