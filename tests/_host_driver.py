"""Build and run a C++ driver of the library's host code (internal headers, linked with the
built library): test infrastructure, no device is touched."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1010_1386_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def run_driver(source, tmp_path):
    """Exit status and standard output of `source`."""
    hipcc = shutil.which("hipcc") or os.path.join(ROCM, "bin", "hipcc")
    clang = os.path.join(ROCM, "llvm", "bin", "clang++")
    if not (os.path.exists(hipcc) and os.path.exists(clang)):
        pytest.skip("ROCm compilers not found")
    src, obj, exe = (str(tmp_path / n) for n in ("driver.cpp", "driver.o", "driver"))
    with open(src, "w") as fh:
        fh.write(source)
    subprocess.run([hipcc, "-std=c++17", "-x", "hip", "--offload-host-only", "-I" + os.path.join(PKG, "csrc"),
                    "-I" + os.path.join(ROOT, "include"), "-c", src, "-o", obj], check=True)
    subprocess.run([clang, obj, "-o", exe, os.path.join(PKG, "librsl.so"), f"-L{ROCM}/lib", "-lamdhip64",
                    f"-Wl,-rpath,{PKG}:{ROCM}/lib"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    return r.returncode, r.stdout
