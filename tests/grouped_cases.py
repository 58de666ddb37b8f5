"""Builds and runs tests/grouped_programs.cpp against the library."""
import os
import subprocess

from paper_2508_01266_amd import lrcc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def run(tmp_path, *args):
    """(exit status, output) of the case named by args."""
    exe = os.path.join(str(tmp_path), "grouped_programs")
    libdir, libname = os.path.split(lrcc.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "paper_2508_01266_amd", "csrc"), "-o", exe,
                    os.path.join(ROOT, "tests", "grouped_programs.cpp"), "-L", libdir, "-l:" + libname,
                    "-Wl,-rpath," + libdir, "-L", os.path.join(ROCM, "lib"), "-lamdhip64",
                    "-Wl,-rpath," + os.path.join(ROCM, "lib")], check=True, timeout=100)
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=60)
    return r.returncode, r.stdout + r.stderr
