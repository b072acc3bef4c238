"""Compile the HIP sources of the library for gfx950 into ``libmoe_mpmc.so`` next to this file, and the Python extension that
marshals its calls' arguments into ``_marshal.so``."""
from __future__ import annotations

import glob
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmoe_mpmc.so")
MARSHAL = os.path.join(HERE, "_marshal.so")            # the Python extension (csrc/marshal.cpp, host code)

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def source_id() -> str:
    """Hash of everything the library is compiled from (csrc/*, include/*.h).  build_library() compiles it
    into the library (moe_build_id()); binding.lib() refuses a library whose id differs from the sources
    beside it, so a stale binary cannot be tested or timed by accident."""
    import hashlib
    h = hashlib.sha256()
    files = sorted(glob.glob(os.path.join(CSRC, "*"))) + sorted(glob.glob(os.path.join(HERE, "..", "include", "*.h")))
    for f in files:
        if os.path.isfile(f):
            h.update(os.path.basename(f).encode() + b"\0")
            h.update(open(f, "rb").read())
    return h.hexdigest()[:16]


def marshal_host() -> str:
    """The torch and the Python whose objects the extension reads through their headers' layout.  build_library() compiles it into the
    extension (built_for); binding.lib() refuses one that was built for others."""
    import sys

    import torch
    return f"torch {torch.__version__} {torch.version.git_version}, python {sys.hexversion >> 24}.{sys.hexversion >> 16 & 255}"


def build_library(verbose: bool = False) -> str:
    """One hipcc -c per source, side by side, then one link; beside them the Python extension."""
    import sysconfig
    from concurrent.futures import ThreadPoolExecutor

    import torch

    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    obj_dir = os.path.join(HERE, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    compile_flags = [f for f in HIPCC_FLAGS if f != "-shared"] + ["-c", f'-DMOE_BUILD_ID="{source_id()}"']

    def run(cmd):
        if verbose:
            print(" ".join(cmd))
        r = subprocess.run(cmd, capture_output=True, text=True)
        msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                         if "packed-fp32-ops" not in l and l.strip())
        if r.returncode != 0:
            raise RuntimeError("the compiler failed:\n" + " ".join(cmd) + "\n" + msgs)
        if verbose and msgs:
            print(msgs)

    srcs = sources()
    objs = [os.path.join(obj_dir, os.path.basename(p)[:-4] + ".o") for p in srcs]
    tdir = os.path.dirname(torch.__file__)
    marshal = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", f'-DMOE_BUILD_ID="{source_id()}"',
               f'-DMOE_BUILT_FOR="{marshal_host()}"', f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I" + os.path.join(tdir, "include"),
               "-I" + os.path.join(tdir, "include", "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
               os.path.join(CSRC, "marshal.cpp"), "-o", MARSHAL, "-L" + os.path.join(tdir, "lib"), "-lc10", "-ltorch_cpu", "-ltorch_python"]
    jobs = min(len(srcs) + 1, max(1, min(8, os.cpu_count() or 1)))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        list(pool.map(run, [marshal] + [[hipcc] + compile_flags + [s, "-o", o] for s, o in zip(srcs, objs)]))
    run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB])
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
