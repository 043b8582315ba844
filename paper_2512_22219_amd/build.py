"""Build libmpk.so (host compiler + HIP runtime) for gfx950, in-tree.

The kernels come in sets (batch class, with or without mixture of experts); csrc/variants.hip is
compiled once per set, in parallel, and the objects are linked with the host side.  Objects go to _build/ next to this file (not committed)."""
import os
import re
import subprocess
import sys
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
         # no packed fp32 instructions: some forms of them have given wrong results now and then
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
_USAGE = "-Rpass-analysis=kernel-resource-usage"   # the compiler says what registers each kernel spills


def variants() -> list:
    """The kernel sets, from their list in kernels.h: dicts with index, nb, moe, level, spills, hybrid_spills."""
    with open(os.path.join(_CSRC, "kernels.h")) as f:
        text = f.read()
    text = text[text.index("#define MPK_VARIANT_LIST"):text.index("#define MPK_COUNT_VARIANT")]
    rows = re.findall(r"X\((\d+), (\d+), (true|false), (O3|Os), (\d+), (\d+)\)", text)
    assert len(rows) == text.count(" X(") and [int(r[0]) for r in rows] == list(range(len(rows))), "MPK_VARIANT_LIST"
    return [dict(index=int(i), nb=int(nb), moe=moe == "true", level="-" + level, spills=int(s), hybrid_spills=int(h))
            for i, nb, moe, level, s, h in rows]


def check_spills(variant: dict, remarks: str) -> None:
    """Raises if a kernel of the set spills more vector registers than its entry in the list allows."""
    found = re.findall(r"Function Name: (\S*mpk_\w+_kernel\S*) .*?VGPRs Spill: (\d+)", remarks, re.S)
    if not found:
        raise RuntimeError(f"kernel set {variant['index']}: the compiler names no kernel's registers")
    for name, spilled in found:
        hybrid = re.search(r"mega_kernelILi\d+ELb[01]ELb1E", name)
        allowed = variant["hybrid_spills" if hybrid else "spills"]
        if int(spilled) > allowed:
            raise RuntimeError(f"kernel set {variant['index']}: {name} spills {spilled} vector registers, {allowed} allowed")


def _compile(job):
    src, obj, extra, variant = job
    r = subprocess.run(["hipcc", *FLAGS, *extra, "-c", src, "-o", obj], stderr=subprocess.PIPE, text=True)
    if not os.environ.get("MPK_BUILD_QUIET"):
        said = r.stderr.splitlines() if r.returncode else [m for m in r.stderr.splitlines() if "warning:" in m]
        sys.stderr.write("".join(m + "\n" for m in said))
    r.check_returncode()
    if variant is not None:
        check_spills(variant, r.stderr)
    return obj


def stale() -> bool:
    """Is a source, or this file with its flags, newer than the library?"""
    return not os.path.exists(LIB) or os.path.getmtime(LIB) < max(map(os.path.getmtime, SOURCES + HEADERS + [os.path.abspath(__file__)]))


def build(force: bool = True, jobs: int = 8) -> str:
    """Compile the library.  force=False rebuilds only when something that it is made from is newer."""
    if not force and not stale():
        return LIB
    os.makedirs(_OBJ, exist_ok=True)
    work = [(SOURCES[0], os.path.join(_OBJ, "compiler.o"), [], None),
            (SOURCES[1], os.path.join(_OBJ, "runtime.o"), [], None)]
    work += [(SOURCES[2], os.path.join(_OBJ, f"variant{v['index']}.o"), [f"-DMPK_VARIANT_INDEX={v['index']}", v["level"], _USAGE], v)
             for v in variants()]
    # the matrix-core sets with experts take longest: start them first
    work.sort(key=lambda j: 0 if j[3] and j[3]["moe"] and j[3]["nb"] in (4, 8, 16) else 1)
    with ThreadPoolExecutor(max_workers=max(1, min(jobs, len(work)))) as pool:
        objs = list(pool.map(_compile, work))
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    return LIB


if __name__ == "__main__":
    print(build())
