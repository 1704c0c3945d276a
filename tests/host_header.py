"""Compiles host-only headers of the library with g++ (no HIP, no GPU) and loads the result with ctypes."""
import ctypes
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23928_amd", "csrc")


def load(source, tmp_path):
    src, so = tmp_path / "host.cpp", tmp_path / "host.so"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, "-o", str(so), str(src)], check=True)
    return ctypes.CDLL(str(so))
