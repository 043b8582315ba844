"""Build libmpk.so (host compiler + HIP runtime) for gfx950, in-tree.

The kernels come in sets (batch class, with or without mixture of experts); csrc/variants.hip is
compiled once per set, in parallel, and the objects are linked with the host side.  Objects go to _build/ next to this file (not committed)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
_CSRC = os.path.join(_HERE, "csrc")
_OBJ = os.path.join(_HERE, "_build")
LIB = os.path.join(_HERE, "libmpk.so")
SOURCES = [os.path.join(_CSRC, f) for f in ("compiler.cpp", "runtime.hip", "variants.hip")]
HEADERS = [os.path.join(_CSRC, "mpk_internal.h"), os.path.join(_CSRC, "kernels.h"),
           os.path.join(os.path.dirname(_HERE), "include", "mpk.h")]
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
         "-I" + os.path.join(os.path.dirname(_HERE), "include"),
         # packed fp32 instructions are not to be generated on this machine pool
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# Kernel sets are compiled for size.  Two compute units share 64 KB of instructions, and a layer of a mixture of experts walks
# through more than that: its instruction cache misses 1300 times a layer at batch 1, 5400 at batch 16 (of some 3500 lines
# that a dense layer is made of and that stay), each a trip to the L2 for a whole workgroup.  us a step, -O3 / -Os: mixture of
# experts at batch 1 688 / 667, batch 16 1396 / 1378; dense sets, which fit, 0 to 2 % (tiny model 34.6 / 34.1, 8B 2690 / 2680, 8B layers at
# batch 8 1002 / 997, 2B class at batch 2, four tokens 2039 / 2027).  Not the set of one packed row (1B class 619 both, shorter rows +0.6 %).
_FOR_SPEED = (11,)


def _n_variants() -> int:
    with open(os.path.join(_CSRC, "kernels.h")) as f:
        return int(re.search(r"kNumVariants\s*=\s*(\d+)", f.read()).group(1))


def _compile(job):
    src, obj, extra = job
    subprocess.check_call(["hipcc", *FLAGS, *extra, "-c", src, "-o", obj],
                          stderr=subprocess.DEVNULL if os.environ.get("MPK_BUILD_QUIET") else None)
    return obj


def build(force: bool = True, jobs: int = 8) -> str:
    """Compile the library.  force=False rebuilds only when a source is newer than the library."""
    if not force and os.path.exists(LIB):
        newest = max(os.path.getmtime(p) for p in SOURCES + HEADERS)
        if os.path.getmtime(LIB) >= newest:
            return LIB
    os.makedirs(_OBJ, exist_ok=True)
    work = [(SOURCES[0], os.path.join(_OBJ, "compiler.o"), []),
            (SOURCES[1], os.path.join(_OBJ, "runtime.o"), [])]
    work += [(SOURCES[2], os.path.join(_OBJ, f"variant{i}.o"), [f"-DMPK_VARIANT_INDEX={i}"] + ([] if i in _FOR_SPEED else ["-Os"]))
             for i in range(_n_variants())]
    # the matrix-core sets with experts take longest: start them first
    work.sort(key=lambda j: 0 if j[1].endswith(("variant8.o", "variant9.o", "variant10.o")) else 1)
    with ThreadPoolExecutor(max_workers=max(1, min(jobs, len(work)))) as pool:
        objs = list(pool.map(_compile, work))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    return LIB


if __name__ == "__main__":
    print(build())
