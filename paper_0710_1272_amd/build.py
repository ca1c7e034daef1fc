"""Builds the gfx950 shared library liblbmd.so from csrc/ with hipcc (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIBDIR = os.path.join(PKG, "_lib")
LIB = os.path.join(LIBDIR, "liblbmd.so")
SOURCES = ["lb_kernels.hip", "md_kernels.hip", "lbmd_api.hip"]
# the bead kernel's variants, each an object of its own: (arithmetic type, periodic axes, polymer model)
BEAD_VARIANTS = [(real, per, poly) for real in ("double", "float") for poly in (1, 0) for per in (1, 0)]
# the one-launch coupled step's variants: (storage, polymer model)
STEP_VARIANTS = [(storage, poly) for poly in (1, 0) for storage in (0, 1, 2, 3)]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed FP32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def build(verbose: bool = False) -> str:
    os.makedirs(LIBDIR, exist_ok=True)
    units = [(s, s.replace(".hip", ".o"), []) for s in SOURCES]
    for real, per, poly in BEAD_VARIANTS:
        units.append(("md_bead.hip", f"md_bead_{real}_{per}{poly}.o",
                      [f"-DMD_REAL={real}", f"-DMD_PERIODIC={per}", f"-DMD_POLY={poly}"]))
    for storage, poly in STEP_VARIANTS:
        units.append(("md_step.hip", f"md_step_{storage}_{poly}.o", [f"-DMD_STORAGE={storage}", f"-DMD_POLY={poly}"]))
    units = [(src, os.path.join(LIBDIR, obj), defs) for src, obj, defs in units]
    objs = [obj for _, obj, _ in units]

    def compile_one(unit):
        src, obj, defs = unit
        cmd = [HIPCC, *FLAGS, *defs, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        out = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{out}")
        if verbose and out.strip():
            print(out, file=sys.stderr)

    with ThreadPoolExecutor(max_workers=min(len(units), 8)) as ex:
        list(ex.map(compile_one, units))
    tmp = LIB + ".tmp"
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
