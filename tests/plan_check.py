"""Compiles a few lines of C++ against the launch-shape rules (csrc/sj_plan.h: plain host arithmetic) and runs them."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def run_program(tmp_path, source):
    """Standard output of a C++ program that includes the rules."""
    src, exe = tmp_path / "plans.cpp", tmp_path / "plans"
    src.write_text('#include "sj_plan.h"\n#include <cstdio>\nusing namespace sj;\n' + source)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_2510_02329_amd", "csrc"), "-o", str(exe), str(src)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout


# d_model, columns of Q + K + V, of Q, FFN width: the shapes of the workloads, then generic ones
SHAPES = [(256, 768, 256, 768), (512, 1536, 1024, 1408), (2048, 3072, 2048, 8192), (4096, 6144, 4096, 14336), (8192, 10240, 8192, 28672),
          (64, 192, 64, 64), (320, 448, 320, 832), (1536, 4608, 1536, 4096), (3072, 5120, 4096, 8128), (5120, 7168, 5120, 13824), (16384, 18432, 16384, 53248)]


def shapes_array():
    return "static const int shapes[][4] = {" + ", ".join("{%d, %d, %d, %d}" % s for s in SHAPES) + "};\n"
