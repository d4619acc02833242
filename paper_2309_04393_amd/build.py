"""Build the gfx950 HIP library libresoct.so in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(HERE, "_lib")
LIB = os.path.join(OUT_DIR, "libresoct.so")
# (source, extra flags); the instantiations of render.hip are compiled in parts
SOURCES = [("render.hip", ["-DRO_PART=4"]), ("render.hip", ["-DRO_PART=3"]), ("render.hip", ["-DRO_PART=2"]),
           ("render.hip", ["-DRO_PART=1"]), ("serve.hip", []), ("api.hip", []), ("render.hip", ["-DRO_PART=0"]),
           ("stream.hip", []), ("octree.hip", []), ("mlp.hip", []), ("prefetch.hip", [])]

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # no packed-FP32 instructions anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False, csrc: str = CSRC, lib: str = LIB) -> str:
    """Compile every source (in parallel) and link lib."""
    out_dir = os.path.dirname(lib)
    os.makedirs(out_dir, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmds, objs = [], []
    for n, (src, extra) in enumerate(SOURCES):
        obj = os.path.join(out_dir, src.replace(".hip", f"_{n}.o"))
        cmds.append([hipcc, *FLAGS, *extra, "-I", os.path.join(ROOT, "include"), "-I", csrc, "-c",
                     os.path.join(csrc, src), "-o", obj])
        objs.append(obj)
    if verbose:
        for c in cmds:
            print(" ".join(c), flush=True)
    jobs = max(1, min(len(cmds), os.cpu_count() or 1, int(os.environ.get("MAX_JOBS", "16"))))
    with ThreadPoolExecutor(jobs) as ex:
        list(ex.map(subprocess.check_call, cmds))
    tmp = lib + ".tmp"
    subprocess.check_call([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", tmp])
    os.replace(tmp, lib)
    return lib


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
