"""Build libcompams.so (HIP kernels + C ABI) for gfx950, in-tree.

`python -m paper_2205_05632_amd.build` compiles every source under csrc/ with hipcc and links
paper_2205_05632_amd/libcompams.so.  Floating-point contraction is off so that every fp32 operation of
the optimizer update rounds once, and packed-fp32 instruction selection is disabled.  A kernel's first plain arguments arrive in
scalar registers (up to the first structure, 14 words), where the first loads of a short kernel would wait for them.  The block-sign
kernels of small steps have what those loads need in front (4 x 65536: 11.9 -> 11.5 us a step), and so have the packing kernels and the
call without a workspace (64 x 300000 in two halves 108.2 -> 107.5, 4 x 300007 43.95 -> 43.8).  The top-k kernels of a context's step have a
structure in front, which switches it off: with plain arguments the one that selects short rows cost a step 0.2 us (4 x 65536: 23.3 ->
23.5), the four of the general route 0.3 (64 x 300000: 90.05 -> 90.35).
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libcompams.so")
SOURCES = ["compams_api.hip", "compams_topk.hip", "compams_blocksign.hip", "compams_wire.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=16",
         "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option"]


def _newer(target, deps):
    if not os.path.exists(target):
        return False
    t = os.path.getmtime(target)
    return all(os.path.getmtime(d) <= t for d in deps)


def build(force: bool = True, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    headers = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    headers.append(os.path.join(os.path.dirname(HERE), "include", "compams.h"))
    objs, jobs = [], []
    for src in SOURCES:
        s = os.path.join(CSRC, src)
        o = os.path.join(OBJ, src.replace(".hip", ".o"))
        objs.append(o)
        if force or not _newer(o, [s] + headers):
            jobs.append([HIPCC] + FLAGS + ["-c", s, "-o", o])

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + r.stdout + r.stderr)
        return r.stderr

    with ThreadPoolExecutor(max_workers=min(4, max(1, len(jobs)))) as ex:
        for warn in ex.map(run, jobs):
            if verbose and warn.strip():
                print(warn)
    if jobs or not os.path.exists(LIB):
        run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB])
    return LIB


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv, verbose=True))
