"""Compiles the launch rules of the library's headers (plain C++ beside the kernels) for the host, for tests that ask them."""
import ctypes
import os
import subprocess

from paper_2602_21233_amd import build


def compile_shim(folder, source):
    (folder / "shim.hip").write_text(source)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", build.CSRC,
                    str(folder / "shim.hip"), "-o", str(folder / "shim.so")], check=True, capture_output=True)
    return ctypes.CDLL(str(folder / "shim.so"))
