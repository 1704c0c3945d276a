"""Builds the HIP library (libhivis.so) in-tree for gfx950 with hipcc."""
import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB_PATH = os.path.join(HERE, "libhivis.so")
SOURCES = [os.path.join(HERE, "csrc", "hivis.hip")]
HEADERS = [os.path.join(HERE, "csrc", n) for n in ("hivis_sizes.h", "hivis_rotary.h", "hivis_kernels.h", "hivis_gemm.h", "hivis_fused.h", "hivis_stream.h", "hivis_tile.h", "hivis_attn.h", "hivis_tree.h")] + [os.path.join(ROOT, "include", "hivis.h")]


def hipcc_path():
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found")
    return p


def build(verbose=True):
    cmd = [hipcc_path(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-shared", "-fPIC",
           # keep the compiler from forming packed-fp32 instructions (hipcc device-pass flag)
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
           "-o", LIB_PATH] + SOURCES
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                    if "packed-fp32-ops" not in l)        # host pass does not know the device feature: harmless
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    return LIB_PATH


if __name__ == "__main__":
    build()
