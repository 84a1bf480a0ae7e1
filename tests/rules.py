"""The library's dispatch rules (csrc/rules.h), compiled for the host: a small
C wrapper around each, called through ctypes."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include "rules.h"
using namespace mlmix;
extern "C" int padded_nrad(int n) { return rules::padded_nrad(n); }
extern "C" int o3_count_first(int scap) { return rules::o3_count_first(scap); }
extern "C" int o3_classes(int ns, int ch, double flops) { return rules::o3_classes(ns, ch, flops); }
extern "C" int o3_split_log(int ntile, int grid, int most, int fill) { return rules::o3_split_log(ntile, grid, most, fill); }
"""


def load(folder):
    src, lib = os.path.join(folder, "rules.cpp"), os.path.join(folder, "librules.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    csrc = os.path.join(ROOT, "paper_2502_19081_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, src, "-o", lib])
    lib = ctypes.CDLL(lib)
    lib.o3_classes.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_double]
    return lib
