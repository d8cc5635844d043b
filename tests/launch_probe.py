"""What libtri.so launches, without a GPU: run as a program with the fake HIP runtime's library (fake_hip.cpp) and a JSON list of
calls, prints for each its status and the runtime's log.  The fake runtime has to be loaded ahead of the real one, hence the process
of its own and the empty stand-in for torch (the binding imports it; nothing here needs it)."""
import ctypes
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ANY = 1 << 20   # an address: nothing is dereferenced


def run(calls):
    """[{"entry": name, sizes and options...}] -> [(status, [(kernel, (x, y, z), threads, lds)], [(kernel, LDS limit)])]"""
    with tempfile.TemporaryDirectory(prefix="fake_hip_") as tmp:
        so = os.path.join(tmp, "libfake_hip.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
        out = subprocess.run([sys.executable, os.path.abspath(__file__), so], input=json.dumps(calls), capture_output=True, text=True,
                             timeout=120)
        assert out.returncode == 0, out.stderr
    result = []
    for status, log in json.loads(out.stdout):
        launches, limits = [], []
        for line in log.splitlines():
            what, name, *numbers = line.split()
            n = [int(x) for x in numbers]
            if what == "limit":
                limits.append((name, n[0]))
            else:
                launches.append((name, tuple(n[:3]), n[3], n[4]))
        result.append((status, launches, limits))
    return result


def call(T, lib, c):
    import numpy as np
    g = c.get
    offsets = np.arange(1, g("offsets", 16) + 1, dtype=np.int64)
    model = T.TriModel(g("layers", 1), g("kv_heads", 1) * g("group", 1), g("kv_heads", 1), 128, 1e6, g("pairs", 0), len(offsets),
                       offsets.ctypes.data_as(ctypes.c_void_p), 0, None)
    n, budget, block = g("n", 1000), g("budget", 100), g("block", 0)
    m = ctypes.byref(model)
    if c["entry"] == "centers":
        return lib.tri_build_centers(m, ANY, g("dtype", 1), g("tokens", 1), ANY, None)
    cache = ctypes.byref(T.TriCache(ANY, ANY, ANY, g("dtype", 1), g("seqs", 1), ANY, ANY, n, block, ANY if block else 0,
                                    -(-n // block) if block else 0, 1 << 12, 1 << 12, 1 << 12, g("stride", 128), 0, 0, 0, g("rotated", 0)))
    if c["entry"] == "select":
        return lib.tri_select_topk(m, ANY + g("offset", 0), cache, budget, ANY, ANY, None, 0, None)
    ws = lib.tri_workspace_size(m, cache, budget)
    if c["entry"] == "score":
        return lib.tri_score(m, ANY, cache, ANY, ANY, ANY, ws, None)
    return lib.tri_compress_step(m, ANY, cache, None if g("fill") else cache, budget, ANY, ANY, ANY, ANY, ws, None)


if __name__ == "__main__":
    import types
    fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
    fake.fake_log.restype = ctypes.c_char_p
    sys.modules["torch"] = types.ModuleType("torch")
    sys.path.insert(0, ROOT)
    from paper_2604_04921_amd import binding
    lib = binding.lib()
    results = []
    for c in json.load(sys.stdin):
        status = call(binding, lib, c)
        results.append((status, fake.fake_log().decode()))
    json.dump(results, sys.stdout)
