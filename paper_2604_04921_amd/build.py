"""Builds libtri.so (the HIP kernels and the C ABI) for gfx950 with hipcc, in-tree."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtri.so")
SOURCES = ["tri_api.hip", "tri_centers.hip", "tri_score.hip", "tri_score_mfma.hip", "tri_select.hip", "tri_compact.hip"]
# (source, flags): the general score kernel's variants, a compilation per group size
UNITS = [("tri_score_lane.hip", ["-DTRI_LANE_GROUP=%d" % g]) for g in (8, 7, 6, 5, 4, 3, 2, 1)] + [(s, []) for s in SOURCES]

# packed fp32 VALU forms are switched off for every kernel of this library
HIPCC_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
               "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc():
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def build(verbose=False, extra=()):
    """Compile every .hip source (in parallel, one hipcc process each) and link libtri.so.  Always recompiles."""
    import tempfile
    from concurrent.futures import ThreadPoolExecutor

    def clean(text):   # hipcc's host pass does not know the packed-fp32 feature name and says so: harmless
        return "\n".join(l for l in text.splitlines() if "packed-fp32-ops" not in l)

    with tempfile.TemporaryDirectory(prefix="libtri_build_") as tmp:
        def compile_one(unit):
            src, flags = unit
            obj = os.path.join(tmp, "%d_%s" % (UNITS.index(unit), src.replace(".hip", ".o")))
            cmd = [hipcc(), *HIPCC_FLAGS, *extra, *flags, "-c", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                   os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            return src, obj, res.returncode, clean(res.stdout)

        with ThreadPoolExecutor(max_workers=min(len(UNITS), os.cpu_count() or 1)) as ex:
            results = list(ex.map(compile_one, UNITS))
        for src, _, rc, out in results:
            if rc != 0:
                raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
            if verbose and out.strip():
                print(out)
        cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", *[r[1] for r in results], "-o", LIB]
        res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if res.returncode != 0:
            raise RuntimeError("link failed:\n" + clean(res.stdout))
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra=sys.argv[1:])
