"""Builds the simulator's shared library in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libgnr_sim.so")
OBJ = os.path.join(HERE, "_build")
# every policy variant of the step kernel is a translation unit of its own, so that they compile side by side
STEP_VARIANTS = ["plain", "rr", "im", "ab", "ab_rr", "ab_im", "ws"]
SOURCES = ["gnr_kernels.hip", "gnr_api.cpp", "gnr_tables.cpp"] + [f"gnr_step_{v}.hip" for v in STEP_VARIANTS]
HEADERS = [os.path.join(CSRC, "gnr_step.h"), os.path.join(CSRC, "gnr_internal.h"), os.path.join(INCLUDE, "gnr_sim.h")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-ffp-contract=off",
         # no packed fp32 instructions in device code (the host pass does not know the feature and says so)
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function",
         # atomics stay one per lane: a few lanes of a wave have something to add as a rule, and where all have the sum is
         # spread over several words. The compiler's rewrite into wave-wide scans costs 60 % with the randomized router (10000
         # servers x 256 replications 6.9 -> 11.0 ms per 300 steps), 46 % with the weighted one (9.0 -> 13.0), 14 % with
         # immediate decode (19.8 -> 22.6 per 2000), 7 % with the convergence instance, 0 to 1 % with the base router
         "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
         # loops are unrolled where the source asks for it (#pragma unroll). Unrolling the others by heuristic too, which the kernel
         # that executed every iteration lost by, changes the timed cases by -0.7 to +0.4 % with this one, which is noise
         "-fno-unroll-loops",
         # the step kernel lives at its register limit: loop strength reduction and the hoisting of loop invariants
         # in machine code both trade registers for instructions, which here ends in spills (sixteen waves: base form 7
         # registers with them and none without, weighted router 28 and 2; two waves dense 6 and none). They cost 3 % with 1024
         # servers x 2048 replications (17.9 -> 18.5 ms per 1000 steps) and with the convergence instance, 4 % with the weighted
         # router (9.0 -> 9.3 per 300), 1 % with 2048 x 1024, nothing with 10000 x 256, and give 1 % with 256 x 1024
         "-mllvm", "-disable-lsr", "-mllvm", "-disable-machine-licm"]


def _compile(src: str, force: bool, verbose: bool) -> str:
    path = os.path.join(CSRC, src)
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    deps = [path] + HEADERS
    if not force and os.path.exists(obj) and all(os.path.getmtime(obj) > os.path.getmtime(d) for d in deps):
        return obj
    cmd = [HIPCC] + FLAGS + [f"-I{INCLUDE}", f"-I{CSRC}", "-c", path, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{out}")
    if out.strip():
        print(out, flush=True)
    return obj


def build(verbose: bool = False, force: bool = True, jobs: int | None = None) -> str:
    """Compiles every source (all of them when `force`, else those older than their object) and links the library."""
    os.makedirs(OBJ, exist_ok=True)
    jobs = jobs or min(len(SOURCES), os.cpu_count() or 1, 16)
    with ThreadPoolExecutor(jobs) as pool:
        objs = list(pool.map(lambda s: _compile(s, force, verbose), SOURCES))
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


def lib_path() -> str:
    """Path of the built library; raises if it has not been built."""
    if not os.path.exists(LIB):
        raise FileNotFoundError(f"{LIB} is missing: run `python -m paper_2602_02987_amd.build` (needs hipcc)")
    return LIB


if __name__ == "__main__":
    import sys
    print(build(verbose=True, force="--changed" not in sys.argv))
