"""Compiles a few lines of C++ against libsj.so and a HIP runtime that only keeps a record (hip_stub.h) and runs them, on the CPU."""
import os
import subprocess

import paper_2510_02329_amd as sj

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_program(tmp_path, source):
    """Standard output of a program; its last line is "0 failures" when every CHECK held."""
    lib = os.environ.get("SJ_TEST_LIB", sj.lib_path())
    if not os.path.exists(lib):
        from paper_2510_02329_amd.build import build_library
        build_library(verbose=False)
    src, exe = tmp_path / "host.cpp", tmp_path / "host"
    src.write_text('#include "hip_stub.h"\n' + source)
    # -rdynamic: the library looks its HIP calls up in the program first
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-rdynamic", "-I", os.path.join(ROOT, "tests"), "-I", os.path.join(ROOT, "include"), "-o", str(exe),
                    str(src), lib, "-Wl,--allow-shlib-undefined", "-Wl,-rpath," + os.path.dirname(lib)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stdout, res.stderr)
    return res.stdout
