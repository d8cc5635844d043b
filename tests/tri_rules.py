"""The score kernels' host-side rules as the library has them: csrc/tri_items.h, compiled by itself."""
import ctypes
import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WRAPPER = """
#include "tri_items.h"
extern "C" {
int item_keys(long long instances, int n, int n_cu) { return tri::item_keys(instances, n, n_cu); }
int large_batch(long long instances, int n, int n_cu) { return tri::large_batch(instances, n, n_cu); }
int sixteen_lane_kernel(int group, long long instances, int n, int n_cu, int half_split, int paged, int rotated)
{
    return tri::sixteen_lane_kernel(group, tri::item_keys(instances, n, n_cu), instances, n, n_cu, half_split, paged, rotated);
}
int stretch_rounds(int group, long long instances, int n, int n_cu) { return tri::stretch_rounds(group, instances, n, n_cu); }
int stretches(int group, long long instances, int n, int n_cu, unsigned total, unsigned longest, int half_split, int paged, int rotated)
{
    const int most = tri::stretch_rounds(group, instances, n, n_cu) * n_cu, entries = tri::stretch_entries(n, tri::stretch_least(instances, n, most));
    return (int)tri::stretches_wanted(total, longest, entries, most, n_cu, tri::lane_waves(group, paged, rotated, half_split));
}
int stretch_seqs(void) { return tri::kStretchSeqs; }
int tile_first(int first, int cnt) { return tri::tile_first(first, cnt); }
int tile_last(int rows, int first, int cnt) { return tri::tile_last(rows, first, cnt); }
}
"""


@functools.lru_cache(maxsize=None)
def library():
    with tempfile.TemporaryDirectory(prefix="tri_rules_") as tmp:
        src, so = os.path.join(tmp, "rules.cpp"), os.path.join(tmp, "rules.so")
        with open(src, "w") as f:
            f.write(WRAPPER)
        subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-shared", "-fPIC",
                        "-I" + os.path.join(ROOT, "paper_2604_04921_amd", "csrc"), src, "-o", so], check=True)
        lib = ctypes.CDLL(so)
    lib.item_keys.argtypes = lib.large_batch.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    lib.stretch_rounds.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    lib.stretches.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_uint, ctypes.c_uint] + [ctypes.c_int] * 3
    lib.sixteen_lane_kernel.argtypes = [ctypes.c_int, ctypes.c_longlong] + [ctypes.c_int] * 5
    return lib


def item_keys(instances, n, n_cu):
    return library().item_keys(instances, n, n_cu)


def large_batch(instances, n, n_cu):
    return bool(library().large_batch(instances, n, n_cu))


def sixteen_lane_kernel(group, instances, n, n_cu, half_split=False, paged=True, rotated=False):
    return bool(library().sixteen_lane_kernel(group, instances, n, n_cu, half_split, paged, rotated))


def score_path(group, instances, n, n_cu, n_seqs, half_split=False, paged=False, rotated=False):
    """How bf16 keys (contiguous, or in blocks of 16 and more) are scored: "sixteen" lanes per key, or by the general kernel in "stretches" or
    work "items"."""
    if sixteen_lane_kernel(group, instances, n, n_cu, half_split, paged, rotated):
        return "sixteen"
    return "stretches" if n_seqs <= library().stretch_seqs() and library().stretch_rounds(group, instances, n, n_cu) > 0 else "items"
