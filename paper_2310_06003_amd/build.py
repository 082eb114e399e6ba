"""Builds libparo.so (host plan + gfx950 kernels) in-tree with hipcc, and the binding's extension with g++."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SO = os.path.join(HERE, "libparo.so")
SOURCES = [os.path.join(HERE, "csrc", "plan.cpp"), os.path.join(HERE, "csrc", "kernels.hip")]
# the extension reads CPython's own structures: its name carries the interpreter that it was built for, so that no other loads it
MARSHAL_SO = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))
MARSHAL_SOURCE = os.path.join(HERE, "csrc", "marshal.cpp")
HEADERS = [os.path.join(HERE, "csrc", h) for h in ("plan.hpp", "device_util.hpp", "loaders.hpp")] + \
          [os.path.join(ROOT, "include", "paro.h")]

# -ffp-contract=off: every fp32 operation of the fold and of Adam is rounded on its own, so
#   results do not depend on which multiply-adds the compiler could fuse.
# -packed-fp32-ops off: scalar fp32 arithmetic only.
# -amdgpu-kernarg-preload-count: the first 14 words of a kernel's arguments are in scalar registers when a wave starts (as many as there
# are), where it would begin with one or two trips to the scalar cache; the kernels take what their first loads need first.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-mllvm", "-amdgpu-kernarg-preload-count=14", "-Wall",
         "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(HERE, "csrc")]
MARSHAL_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
                 "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"]]

STAMP = SO + ".srchash"        # hash of what the library in the tree was built from


def source_hash() -> str:
    """sha256 over the compiler flags, the interpreter's ABI and the text of every source and header."""
    flags = FLAGS[:-2] + MARSHAL_FLAGS[:-2]                         # without the -I paths (they differ per checkout)
    h = hashlib.sha256(" ".join(flags + [sysconfig.get_config_var("EXT_SUFFIX")]).encode())
    for f in SOURCES + [MARSHAL_SOURCE] + HEADERS:
        h.update(os.path.basename(f).encode())
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def built_hash() -> str:
    """The source hash recorded when the library in the tree was built ("" if unknown)."""
    try:
        with open(STAMP) as fh:
            return fh.read().strip()
    except OSError:
        return ""


def stale() -> bool:
    """True when there is no library, or it was built from other sources than the tree holds."""
    return not (os.path.exists(SO) and os.path.exists(MARSHAL_SO)) or built_hash() != source_hash()


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if os.path.exists(STAMP):
        os.remove(STAMP)
    for cmd in ([hipcc] + FLAGS + SOURCES + ["-o", SO],
                [os.environ.get("CXX", "g++")] + MARSHAL_FLAGS + [MARSHAL_SOURCE, "-o", MARSHAL_SO]):
        if verbose:
            print(" ".join(cmd))
        subprocess.run(cmd, check=True)
    with open(STAMP, "w") as fh:
        fh.write(source_hash() + "\n")
    return SO


if __name__ == "__main__":
    build(verbose=True)
