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
extern "C" int o3_order_span(int n, int blocks) { return rules::o3_order_span(n, blocks); }
extern "C" int o3_classes(int ns, int ch, double flops) { return rules::o3_classes(ns, ch, flops); }
extern "C" int o3_split_log(int ntile, int grid, int most, int fill) { return rules::o3_split_log(ntile, grid, most, fill); }
extern "C" double o3_weight(int form, int reduced, int classes, double sparse, double dense)
{ return rules::o3_weight(form, reduced, classes, sparse, dense); }
extern "C" int fork_after_basis(int form, double w, int n, int rebuild) { return rules::fork_after_basis(form, w, n, rebuild); }
"""


def load(folder):
    src, lib = os.path.join(folder, "rules.cpp"), os.path.join(folder, "librules.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    csrc = os.path.join(ROOT, "paper_2502_19081_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I", csrc, src, "-o", lib])
    lib = ctypes.CDLL(lib)
    lib.o3_classes.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_double]
    d, i = ctypes.c_double, ctypes.c_int
    lib.o3_weight.argtypes, lib.o3_weight.restype = [i, i, i, d, d], d
    lib.fork_after_basis.argtypes = [i, d, i, i]
    return lib
