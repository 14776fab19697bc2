"""Build libsmre.so (HIP, gfx950) in-tree with hipcc."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsmre.so")
SOURCES = [os.path.join(CSRC, "smre.hip"), os.path.join(CSRC, "phase.hip")]
HEADERS = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hpp", ".h"))] + [
    os.path.join(ROOT, "include", "smre.h")]

FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    "-ffp-contract=off",
    # keep the compiler from emitting packed FP32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]

# Objects: the sweep kernel once per type and region side (longest first), and
# the rest.
TYPES = [("double", "double", "false"), ("float", "float", "true"), ("float", "float", "false"),
         ("float", "bf16_t", "true"), ("float", "bf16_t", "false")]
UNITS = [(SOURCES[1], [f"-DSMRE_TX={tx}", f"-DSMRE_TQ={tq}", f"-DSMRE_KAHAN={ka}", f"-DSMRE_R={r}"])
         for r in (32, 16, 8) for tx, tq, ka in TYPES]
UNITS.insert(len(TYPES), (SOURCES[0], []))


def build(verbose: bool = False) -> str:
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, f"u{i}.o") for i in range(len(UNITS))]
        cmds = [["hipcc"] + FLAGS + defs + ["-c", src, "-o", obj]
                for (src, defs), obj in zip(UNITS, objs)]
        cmds.append(["hipcc", "--offload-arch=gfx950", "-shared"] + objs + ["-o", LIB + ".tmp"])
        if verbose:
            for cmd in cmds:
                print(" ".join(cmd), flush=True)
        jobs = max(1, min(16, len(os.sched_getaffinity(0))))
        with ThreadPoolExecutor(jobs) as pool:
            list(pool.map(subprocess.check_call, cmds[:-1]))
        subprocess.check_call(cmds[-1])
    os.replace(LIB + ".tmp", LIB)
    return LIB


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(f) > t for f in SOURCES + HEADERS)


if __name__ == "__main__":
    build(verbose=True)
