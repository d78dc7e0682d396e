"""Builds libmergecomp.so (the C-ABI HIP library) in-tree with hipcc for gfx950, and _fastcall (the binding's hot calls) with the
host compiler, if there is one and it finds Python's headers: the binding does without it."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
import warnings

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmergecomp.so")
FASTCALL = os.path.join(HERE, "_fastcall" + sysconfig.get_config_var("EXT_SUFFIX"))      # (other interpreters' layouts differ: none but this one loads it)
SOURCES = ["mc_api.hip", "kernels_dense.hip", "kernels_sparse.hip"]

# -ffp-contract=off: the residual updates must round every fp32 operation on its own
# (no fused multiply-add), or codes and residuals would not be reproducible bit for bit.
# packed fp32 instructions are switched off on purpose for this target.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-command-line-argument",
]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32 target feature: harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + out)
    if verbose and out.strip():
        print(out)


def build_fastcall(verbose: bool = False) -> bool:
    """The extension module; without it, a warning and False."""
    untagged = os.path.join(os.path.dirname(FASTCALL), "_fastcall.so")          # (which any interpreter would load)
    if os.path.exists(untagged):
        os.remove(untagged)
    try:
        _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I" + sysconfig.get_paths()["include"],
              "-o", FASTCALL, os.path.join(CSRC, "fastcall.cpp")], verbose)
    except (OSError, RuntimeError) as e:
        if os.path.exists(FASTCALL):             # (of other sources than the library's)
            os.remove(FASTCALL)
        warnings.warn(f"{os.path.basename(FASTCALL)} was not built, all calls go through ctypes: {e}")
        return False
    return True


def build(verbose: bool = False) -> str:
    _run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + HIPCC_FLAGS + ["-o", LIB] + [os.path.join(CSRC, s) for s in SOURCES], verbose)
    build_fastcall(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
