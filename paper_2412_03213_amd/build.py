"""Build libclusterkv.so (gfx950) in-tree with hipcc, and the _ckhost module (the native form of
the binding's hot call, for the interpreter that runs this) with the host compiler.

    python -m paper_2412_03213_amd.build [--force]

Objects go to _build/ at the repository root, the libraries next to this file.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJ_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libclusterkv.so")
HOST_SRC = os.path.join(CSRC, "host_call.cpp")
HOST_LIB = os.path.join(PKG, "_ckhost" + sysconfig.get_config_var("EXT_SUFFIX"))

SOURCES = ["api.hip", "kmeans_assign.hip", "kmeans_assign_stream.hip", "kmeans_assign_wide.hip",
           "kmeans_update.hip", "kmeans_small.hip", "select_gather.hip",
           "sparse_attn.hip", "evaluate.hip", "cluster_cache.hip",
           "probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         # packed-FP32 instruction selection is kept off for every device function
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", INCLUDE, "-I", CSRC]


# per-file additions: keep MFMA accumulators in vector registers where the kernel reads
# them with vector instructions and has other data (MFMA-only operands) for the AGPRs
EXTRA_FLAGS = {f: ["-mllvm", "-amdgpu-mfma-vgpr-form"]
               for f in ("kmeans_assign_stream.hip", "kmeans_assign_wide.hip")}


def _newer(a: str, b: str) -> bool:
    return not os.path.exists(b) or os.path.getmtime(a) > os.path.getmtime(b)


def build(force: bool = False, verbose: bool = True) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hpp")]
    headers.append(os.path.join(INCLUDE, "clusterkv.h"))
    jobs = []
    objs = []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
        objs.append(o)
        if force or _newer(s, o) or any(_newer(h, o) for h in headers):
            jobs.append([HIPCC, *FLAGS, *EXTRA_FLAGS.get(src, []), "-c", s, "-o", o])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"{os.path.basename(cmd[0])} failed:\n{r.stdout}\n{r.stderr}")
        noise = "is not a recognized feature"
        err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
        if verbose and err.strip():
            print(err, flush=True)

    with ThreadPoolExecutor(max_workers=min(4, max(1, len(jobs)))) as ex:
        list(ex.map(run, jobs))
    if force or jobs or not os.path.exists(LIB):
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    header = os.path.join(INCLUDE, "clusterkv.h")
    if force or _newer(HOST_SRC, HOST_LIB) or _newer(header, HOST_LIB):
        # the binding does without it: a machine without a host compiler or Python's headers
        # still gets the library
        if os.path.exists(HOST_LIB):
            os.remove(HOST_LIB)
        try:
            run([CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", INCLUDE,
                 "-I", sysconfig.get_paths()["include"], HOST_SRC, "-o", HOST_LIB])
        except (RuntimeError, OSError) as e:
            print(f"_ckhost is not built, decode_step is called through ctypes: {e}", flush=True)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
