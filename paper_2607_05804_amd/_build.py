"""Build paper_2607_05804_amd/libturnkl.so (the fused turn-KL library) for gfx950."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
SOURCES = ["turnkl_api.hip", "segment.hip", "rowkl.hip", "rowkl_ragged.hip", "rowkl_whole.hip",
           "rowfwd.hip", "reduce.hip", "topk.hip", "controller.cpp", "diagnostics.cpp"]
LIB = os.path.join(HERE, "libturnkl.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed for libturnkl.so")


def build(verbose: bool = False, extra=()) -> str:
    """Compile every source on its own, eight at a time, and link them."""
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory() as d:
        objs = [os.path.join(d, s + ".o") for s in SOURCES]
        cmds = [[HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, s), "-o", o]
                for s, o in zip(SOURCES, objs)]
        with ThreadPoolExecutor(8) as pool:
            list(pool.map(lambda c: _run(c, verbose), cmds))
        _run([HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", *extra, *objs, "-o", tmp], verbose)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
