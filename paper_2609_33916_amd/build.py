"""Build the HIP library libattn_mi355x.so in-tree with hipcc for gfx950, and the
Python binding's native part with g++.

Usage: python -m paper_2609_33916_amd.build [-v]
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
import tempfile
import warnings

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
REPO_DIR = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(REPO_DIR, "include")
LIB_NAME = "libattn_mi355x.so"
LIB_PATH = os.path.join(PKG_DIR, LIB_NAME)
# the entry points' native Python form (host code, against the installed torch)
BINDING_PATH = os.path.join(PKG_DIR, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))
# translation units and their own flags: the bf16 dQ kernel is scheduled
# with the iterative ILP strategy (measured on n = 16384, d = 128 causal: dQ
# 2-4 % faster); the forward (3 % slower under it) and the bf16 dK/dV kernel
# (2 % slower with its 32- and 48-key waves) keep the default strategy
SOURCES = {
    "attn.hip": [],
    "dkdv.hip": [],
    "split.hip": [],
    "f32x3.hip": [],
    "bwd.hip": ["-mllvm", "-amdgpu-sched-strategy=iterative-ilp"],
}

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-mcode-object-version=5",
    # keep the compiler from forming packed FP32 VALU instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA accumulators in arch VGPRs: the softmax reads and rescales them
    # with VALU instructions, which cannot address AGPRs; the AGPR form
    # costs accvgpr copies every key tile
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (expected /opt/rocm/bin/hipcc)")


def binding_command(out: str) -> list:
    import torch
    from torch.utils.cpp_extension import include_paths
    libdir = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = [shutil.which("g++") or "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"]
    cmd += [a for d in (*include_paths(), sysconfig.get_paths()["include"]) for a in ("-isystem", d)]
    return cmd + [os.path.join(CSRC, "binding.cpp"), "-L", libdir, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10",
                  "-o", out]


def build(verbose: bool = False, out: str = LIB_PATH, extra_flags=(), csrc: str = CSRC) -> str:
    """Compile the library and the binding (always recompiles) and return the library's path. ``csrc``
    may name another copy of the sources (variant builds). Each source is
    compiled to an object with its own flags (in parallel), then linked."""
    tmpdir = tempfile.mkdtemp(prefix=".attn_build_", dir=os.path.dirname(os.path.abspath(out)))
    try:
        procs = []
        for src, flags in SOURCES.items():
            obj = os.path.join(tmpdir, src + ".o")
            cmd = [hipcc(), *HIPCC_FLAGS, *flags, *extra_flags, "-I", INCLUDE, "-I", csrc,
                   "-c", os.path.join(csrc, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            procs.append((obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        binding = None
        if out == LIB_PATH:   # variant builds of the library share the package's binding
            cmd = binding_command(os.path.join(tmpdir, "binding.so"))
            if verbose:
                print(" ".join(cmd), flush=True)
            binding = subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        objs = []
        for obj, p in procs:
            _check(p.communicate()[0], p.returncode, verbose)
            objs.append(obj)
        if binding is not None:
            log = binding.communicate()[0]
            bound = binding.returncode == 0
            if not bound:   # the package runs without it, through the Python form of the calls
                warnings.warn(f"the native binding was not built, calls will take the slower Python form:\n{log}",
                              RuntimeWarning)
            elif verbose and log.strip():
                print(log)
        tmp = out + ".tmp"
        cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        _check(res.stdout + res.stderr, res.returncode, verbose)
        os.replace(tmp, out)
        if binding is not None and bound:
            os.replace(os.path.join(tmpdir, "binding.so"), BINDING_PATH)
        elif binding is not None and os.path.exists(BINDING_PATH):
            os.remove(BINDING_PATH)   # of an earlier build
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return out


def _check(output: str, returncode: int, verbose: bool) -> None:
    log = "\n".join(l for l in output.splitlines() if "packed-fp32-ops" not in l)
    if returncode != 0:
        raise RuntimeError(f"hipcc failed ({returncode}):\n{log}")
    if verbose and log.strip():
        print(log)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
