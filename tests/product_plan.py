"""The library's own rule of which kernel takes a linear layer of the separate kernels (csrc/product_plan.h), built for the host."""
import ctypes
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_19131_amd", "csrc")
QKV, PROJ, FC1, FC2 = range(4)
NAMES = ("few", "ring64", "ring128", "tile")

_SOURCE = r'''
#include "product_plan.h"
extern "C" int form(int epi, int rows, int N, int K) { return mixaq::product_form(epi, rows, N, K); }
'''


def _build():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(_SOURCE)
        subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC, "-o", so, src], check=True)
        return ctypes.CDLL(so)


lib = _build()


def form(epi, rows, N, K):
    return NAMES[lib.form(epi, rows, N, K)]


def rows(spec, k_high):
    """Rows of the gathered activations: both regions in whole 128s."""
    region = lambda windows: -(-spec.B * windows * 49 // 128) * 128
    return region(k_high) + region(spec.nW - k_high)


def forms(spec, k_high):
    """The kernels of the projection, FC1 and FC2 of such a block."""
    R, C, F = rows(spec, k_high), spec.C, spec.C * spec.mlp_ratio
    return form(PROJ, R, C, C), form(FC1, R, F, C), form(FC2, R, C, F)
