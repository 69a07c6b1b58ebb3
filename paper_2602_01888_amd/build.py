"""Builds libtomg.so (HIP, gfx950) in place with hipcc."""

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtomg.so")
SOURCES = ["api.hip", "kernels.hip", "fused.hip", "tile.hip",
           "march.hip", "tail.hip"]
# the three forms of the level passes, compiled apart, make one object
# (fused.hip.o): none is of use without the others
FORMS = ["fused.hip", "tile.hip", "march.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LLD = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "ld.lld")
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    # packed FP32 instructions stay off on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
    "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"),
    "-I", CSRC,
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def build(verbose: bool = False) -> str:
    """Compiles every source to an object (in parallel), joins the forms of the
    level passes, then links the shared library."""
    from concurrent.futures import ThreadPoolExecutor
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def one(src):
        name = os.path.basename(src)
        obj = os.path.join(objdir, name + (".part.o" if name in FORMS else ".o"))
        cmd = [HIPCC] + compile_flags + ["-c", "-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(one, sources()))
    parts = [o for o in objs if o.endswith(".part.o")]
    fused = os.path.join(objdir, "fused.hip.o")
    cmd = [LLD, "-r", "-o", fused] + parts
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    objs = [o for o in objs if o not in parts] + [fused]
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB + ".tmp"] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = sources() + [os.path.join(CSRC, "tomg_internal.h"), os.path.join(CSRC, "quad.h"),
                        os.path.join(ROOT, "include", "tomg.h")]
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
