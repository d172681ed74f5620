"""Compiles and runs a small host program against the library's internal headers
(CPU only; HIP calls that a header makes inline are defined by the program)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_host(source, tmp_path):
    """stdout of the program `source` (C++17, internal headers on the include path)."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("no host compiler or HIP headers")
    cpp, exe = tmp_path / "prog.cpp", tmp_path / "prog"
    cpp.write_text(source)
    subprocess.run([cxx, "-std=c++17", "-O1", "-w", "-D_GLIBCXX_ASSERTIONS", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2507_21236_amd", "csrc"), "-I", "/opt/rocm/include",
                    str(cpp), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
