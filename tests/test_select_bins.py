"""Where the selection's bins begin (csrc/tri_bins.h, no GPU needed): the least float of every bin, checked against the place of that float
and of the one below it as the kernel computes them."""
import ctypes
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WRAPPER = """
#include <math.h>
#include "tri_bins.h"
extern "C" int wrong_bins(int *first)
{
    int wrong = 0;
    for (int bin = 2047; bin >= 1; --bin) {
        const double edge = tri::bin_edge(bin);
        float f = (float)edge;
        if ((double)f < edge) f = nextafterf(f, INFINITY);
        const float below = nextafterf(f, -INFINITY);
        if (!(fmaf(f, 128.0f, 512.0f) >= (float)bin && fmaf(below, 128.0f, 512.0f) < (float)bin)) ++wrong, *first = bin;
    }
    return wrong;
}
"""


def test_the_least_score_of_every_bin(tmp_path):
    src, so = str(tmp_path / "b.cpp"), str(tmp_path / "b.so")
    with open(src, "w") as f:
        f.write(WRAPPER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I" + os.path.join(ROOT, "paper_2604_04921_amd", "csrc"),
                    src, "-o", so], check=True)
    first = ctypes.c_int(0)
    assert ctypes.CDLL(so).wrong_bins(ctypes.byref(first)) == 0, first.value
