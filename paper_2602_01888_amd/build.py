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
OBJDIR = os.path.join(HERE, "_build")
HEADERS = [os.path.join(CSRC, "tomg_internal.h"), os.path.join(CSRC, "quad.h"),
           os.path.join(ROOT, "include", "tomg.h")]
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


def object_of(name):
    """The object a source is compiled to."""
    return os.path.join(OBJDIR, name + (".part.o" if name in FORMS else ".o"))


def linker():
    """The linker that goes with the compiler in use."""
    out = subprocess.run([HIPCC, "-print-prog-name=ld.lld"], check=True, capture_output=True,
                         text=True)
    return out.stdout.strip()


def build(verbose: bool = False) -> str:
    """Compiles every source to an object (in parallel), joins the forms of the
    level passes, then links the shared library."""
    from concurrent.futures import ThreadPoolExecutor
    os.makedirs(OBJDIR, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def one(src):
        obj = object_of(os.path.basename(src))
        cmd = [HIPCC] + compile_flags + ["-c", "-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(one, sources()))
    parts = [object_of(s) for s in FORMS]
    fused = os.path.join(OBJDIR, "fused.hip.o")
    cmd = [linker(), "-r", "-o", fused] + parts
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


def _older(path, deps):
    return not os.path.exists(path) or any(
        os.path.getmtime(d) > os.path.getmtime(path) for d in deps)


def stale() -> bool:
    return _older(LIB, sources() + HEADERS)


def stale_objects() -> bool:
    """Whether an object is missing or older than what it was made from: code
    that links the objects by hand has to build first then."""
    if any(_older(object_of(s), [os.path.join(CSRC, s)] + HEADERS) for s in SOURCES):
        return True
    return _older(os.path.join(OBJDIR, "fused.hip.o"), [object_of(s) for s in FORMS])


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
