"""Build libsse.so (all HIP sources under csrc/) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import glob
import hashlib
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libsse.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 arithmetic stays off: the compiler may not emit v_pk_* fp32 ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def source_files():
    """Every file the library is built from (kernels, their headers, the ABI header)."""
    return sources() + sorted(glob.glob(os.path.join(HERE, "csrc", "*.h"))) + [os.path.join(ROOT, "include", "sse.h")]


def source_hash() -> str:
    """sha256 over the sources, recorded next to the library when it is built."""
    h = hashlib.sha256()
    for f in source_files():
        h.update(os.path.relpath(f, ROOT).encode())
        with open(f, "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def build(verbose: bool = False, extra=()) -> str:
    """Compile every source and link the library.  The sources compile side by side, the
    largest first: one after another they take eight minutes, most of it in the instances
    of two kernels."""
    digest = source_hash()
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(HERE, "csrc")]
    msgs = []

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        text = "\n".join(l for l in (res.stdout + res.stderr).splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError(f"hipcc failed ({res.returncode}):\n{text}")
        msgs.append(text)

    with tempfile.TemporaryDirectory() as tmp:
        srcs = sorted(sources(), key=lambda f: "kspace" not in f)
        objs = [os.path.join(tmp, os.path.basename(f) + ".o") for f in srcs]
        jobs = min(len(srcs), int(os.environ.get("MAX_JOBS", 0)) or os.cpu_count() or 1, 16)
        with ThreadPoolExecutor(jobs) as pool:
            list(pool.map(lambda so: run([HIPCC, *FLAGS, *extra, *inc, "-c", so[0], "-o", so[1]]), zip(srcs, objs)))
        run([HIPCC, "--offload-arch=gfx950", "-fPIC", "-shared", *extra, *objs, "-o", LIB + ".tmp"])
    if verbose and any(m.strip() for m in msgs):
        print("\n".join(m for m in msgs if m.strip()))
    os.replace(LIB + ".tmp", LIB)
    with open(LIB + ".sha256", "w") as fh:
        fh.write(digest + "\n")
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
