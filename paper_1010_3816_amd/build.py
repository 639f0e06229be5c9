"""Compile libteuk.so for gfx950 with hipcc (in-tree, no JIT cache)."""
import os
import subprocess

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libteuk.so")
SOURCES = ["lw_kernels.hip", "adjoint_kernels.hip", "spin_tangent.hip", "tables.hip",
           "teuk_api.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -packed-fp32-ops: no packed FP32 instructions are generated (all arithmetic
# here is FP64 anyway).  -ffp-contract=on: a multiply and an add are fused
# only within one source expression, never across statements, so code shared
# by several kernels rounds the same way in each of them (the one-step,
# two-step and batched kernels give bit-identical results).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-ffp-contract=on",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd):
    print("+", " ".join(cmd), flush=True)
    r = subprocess.run(cmd, cwd=PKG, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    msg = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if noise not in l)
    if msg.strip():
        print(msg, flush=True)
    if r.returncode != 0:
        raise subprocess.CalledProcessError(r.returncode, cmd)


def build(extra=(), out=None, source_flags=None):
    """Compile every source to an object (source_flags: {source: its own flags}), link the library."""
    lib = out or LIB
    per = source_flags or {}
    objs = []
    for s in SOURCES:
        obj = f"{lib}.{os.path.splitext(s)[0]}.o"
        _run([HIPCC, *FLAGS, *extra, *per.get(s, []), "-x", "hip", "-c", os.path.join(CSRC, s), "-o", obj])
        objs.append(obj)
    tmp = lib + ".tmp"
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
    for o in objs:
        os.remove(o)
    os.replace(tmp, lib)
    return lib


if __name__ == "__main__":
    build()
