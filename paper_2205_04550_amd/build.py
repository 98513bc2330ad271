"""Build libtumordb.so (HIP, gfx950) in place: ``python -m paper_2205_04550_amd.build``."""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libtumordb.so")

SOURCES = ["api.cpp", "pack.hip", "scan.hip", "select.hip", "batch.hip", "nn.hip", "embed.hip",
           "resample.hip", "sparse.hip", "hash.hip", "vae.hip", "noalloc.hip", "knn.hip",
           "train.hip"]
# Sources with floating-point arithmetic that may be contracted into FMAs.
CONTRACT_OK = {"nn.hip", "train.hip"}

HIPCC = os.environ.get("HIPCC", "hipcc")
COMMON = ["--offload-arch=gfx950", "-O3", "-fPIC", "-std=c++17", "-Wall",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
# The Dice arithmetic is IEEE double and must not be contracted or relaxed.
EXACT = ["-ffp-contract=off", "-fno-fast-math"]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    fp = ["-ffp-contract=fast"] if src in CONTRACT_OK else EXACT
    cmd = [HIPCC, *COMMON, *fp, *lang, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compiling {src} failed:\n{r.stdout}\n{r.stderr}")
    noise = [l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip()]
    if noise and verbose:
        print("\n".join(noise), flush=True)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
