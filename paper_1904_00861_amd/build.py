"""Build libdtsph.so (gfx950) in-tree with hipcc.

Every translation unit is compiled with packed-FP32 instruction selection
disabled; the kernels use ordinary scalar float arithmetic.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libdtsph.so")
# (source, object, extra flags); the pair pass's many variants compile as one
# object per pass type and dimension so that they build in parallel
UNITS = [("dtsph_pair.hip", f"dtsph_pair_{name}{dim}.o", [f"-DDTSPH_PAIR_T={t}", f"-DDTSPH_PAIR_DIM={dim}"])
         for name, t in (("f", "float"), ("d", "double")) for dim in (2, 3)]
UNITS += [(s, s.replace(".hip", ".o"), []) for s in ("dtsph_tail.hip", "dtsph_pass.hip", "dtsph_cells.hip", "dtsph_api.hip")]
ARCH = os.environ.get("DTSPH_ARCH", "gfx950")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", INCLUDE, "-I", CSRC, "-Wall", "-Wno-unused-function",
]


def _compile(src: str, obj: str, extra: list) -> None:
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    noise = [ln for ln in r.stderr.splitlines() if "packed-fp32-ops" not in ln and ln.strip()]
    if noise:
        sys.stderr.write("\n".join(noise) + "\n")


def build(verbose: bool = False) -> str:
    """Compile every source and link libdtsph.so; always rebuilds."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, o) for _, o, _ in UNITS]
    with cf.ThreadPoolExecutor(max_workers=min(8, len(UNITS))) as ex:
        list(ex.map(_compile, [u[0] for u in UNITS], objs, [u[2] for u in UNITS]))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
