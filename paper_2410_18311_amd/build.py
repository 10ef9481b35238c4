"""Builds libcoreinfer.so in-tree with hipcc for gfx950 (cross-compiles
without a GPU).  `python -m paper_2410_18311_amd.build` rebuilds."""

from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

from . import isa_check

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD_DIR = os.path.join(PKG_DIR, "_build")
LIB_PATH = os.path.join(PKG_DIR, "libcoreinfer.so")
# a Python module for this interpreter, linked against the library beside it
BINDING_PATH = os.path.join(PKG_DIR, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))

SOURCES = ["api.hip", "ffn_decode.hip", "ffn_decode_small.hip", "ffn_decode_fused.hip", "ffn_union.hip", "select.hip", "compact.hip", "centroid.hip", "gemv.hip", "gemm_mfma.hip", "gemm_f32.hip", "gemm_wide.hip", "gemm_mid.hip", "gemm_slim_f16.hip", "gemm_slim_bf16.hip", "stream_probe.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", INCLUDE, "-I", CSRC,
]
# development builds: CI_EXTRA_FLAGS="-DCI_FUSED_STAMPS" adds time stamps to the single-launch decode
FLAGS += os.environ.get("CI_EXTRA_FLAGS", "").split()


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, src.replace(".hip", ".o"))
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build_binding() -> bool:
    """The per-token call's C module.  Where there is no C compiler or no Python.h the library serves without it, through ctypes."""
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-shared", "-fPIC", "-I", sysconfig.get_paths()["include"], "-I", INCLUDE,
           os.path.join(CSRC, "binding.c"), "-o", BINDING_PATH, "-L", PKG_DIR, "-lcoreinfer", "-Wl,-rpath,$ORIGIN"]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
        why = r.stderr if r.returncode != 0 else None
    except OSError as e:
        why = str(e)
    if why is None:
        return True
    if os.path.exists(BINDING_PATH):
        os.remove(BINDING_PATH)   # of another library
    sys.stderr.write("no C module for the per-token call, which goes through ctypes instead (0.4 to 1 us more):\n" + why + "\n")
    return False


def build_library(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB_PATH]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    bad = isa_check.hazards(LIB_PATH)
    if bad:
        os.remove(LIB_PATH)
        raise RuntimeError("loads into LDS or matrix products that read a register too soon after it was written, or a product's result read too soon:\n" +
                           "\n".join(bad))
    build_binding()
    if verbose:
        print("built", LIB_PATH)
    return LIB_PATH


if __name__ == "__main__":
    build_library(verbose=True)
