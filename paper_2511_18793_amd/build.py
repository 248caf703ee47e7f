"""Compile the HIP sources into paper_2511_18793_amd/libnezha.so for gfx950."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
# (source, object name, extra flags); the slowest first
UNITS = [("beam.hip", "beam_%d" % k, ["-DBEAM_KST=%d" % k]) for k in (8, 4, 3, 2, 1, 32, 16)]
UNITS += [("draft.hip", "draft", []), ("itemset.hip", "itemset", [])]
OUT = os.path.join(HERE, "libnezha.so")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
         # packed fp32 instructions off: hipcc must not form v_pk_*_f32 from float code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-command-line-argument"]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + err)
    if verbose and err.strip():
        print(err, flush=True)


def build(verbose=False):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    objs = [os.path.join(OBJ, name + ".o") for _, name, _ in UNITS]
    with ThreadPoolExecutor(min(len(UNITS), os.cpu_count() or 1)) as pool:
        jobs = [pool.submit(_run, [hipcc] + FLAGS + extra +
                            ["-c", os.path.join(CSRC, src), "-o", obj], verbose)
                for (src, _, extra), obj in zip(UNITS, objs)]
        for j in jobs:
            j.result()
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", OUT], verbose)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
