"""Builds libamph.so (the HIP kernels and the C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libamph.so")
SOURCES = ["gemv.hip", "draft_mm.hip", "small.hip", "gemm_skinny.hip", "verify_attn.hip", "amph_api.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         # packed-fp32 VALU forms are kept off on the test machines
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


DIGEST = os.path.join(HERE, "_build", "sources.sha256")


def sources_digest() -> str:
    """Of everything under csrc, the C header and the flags."""
    h = hashlib.sha256(" ".join(FLAGS).encode())
    header = os.path.join(HERE, "..", "include", "amph.h")
    for path in sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC)) + [header]:
        with open(path, "rb") as f:
            h.update(os.path.basename(path).encode() + f.read())
    return h.hexdigest()


def built_from() -> str | None:
    """The digest of the sources that the objects in _build were compiled from; None without a finished build."""
    if not os.path.exists(DIGEST):
        return None
    with open(DIGEST) as f:
        return f.read()


def build_library(verbose: bool = True, jobs: int = 6) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    digest = sources_digest()
    if os.path.exists(DIGEST):
        os.remove(DIGEST)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        while len([p for _, p in procs if p.poll() is None]) >= jobs:
            procs[0][1].wait()
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "not a recognized feature" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out, file=sys.stderr)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout)
    with open(DIGEST, "w") as f:
        f.write(digest)
    return LIB


if __name__ == "__main__":
    print(build_library())
