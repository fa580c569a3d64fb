"""Builds librouterelay.so for gfx950 with hipcc (in-tree, next to this file).

Each HIP source is compiled to an object under ``_build/`` in parallel and the
objects are linked into ``paper_2609_07306_amd/librouterelay.so``.  Packed
binary32 VALU instructions are disabled (``-packed-fp32-ops``); device
code is compiled with ``-fno-honor-nans``.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "librouterelay.so")
SOURCES = ["rr_api.hip", "rr_route.hip", "rr_rescore.hip", "rr_rescore_dense.hip", "rr_consumer.hip"] + [
    f"rr_route_{t}_{m}.hip" for t in ("f32", "bf16") for m in ("full", "anchor", "reroute", "relay")]
# the resident-score kernel: one object per caller, input type and width, all from
# rr_resident_inst.hip; each is listed under the name its object takes
RESIDENT = {f"rr_resident_inst_{mode}_{dt}_{d}.hip": (f"-DRR_MODE={mode}", f"-DRR_DT={dt}", f"-DRR_D={d}")
            for mode in ("MODE_FULL", "MODE_ANCHOR", "MODE_RELAY")
            for dt, widths in (("float", (32, 64, 128)), ("bf16_t", (32, 64, 128, 256))) for d in widths}
SOURCES += RESIDENT
# ... whose atomics come from one lane per wave or from lanes with different
# addresses: the compiler's wave-level aggregation would only add a wait for the
# returned value right behind each of them
NO_ATOMIC_OPT = ("-mllvm", "-amdgpu-atomic-optimizer-strategy=None")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-Wall",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no device code relies on what the compiler makes of a NaN (where one may be
    # met, the resident tile's collection, it uses compare and max instructions
    # of its own), so min / max / med3 need no NaN canonicalisation
    "-Xarch_device", "-fno-honor-nans",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(name: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(name)[0] + ".o")
    src, more = name, ()
    if name in RESIDENT:
        src, more = "rr_resident_inst.hip", RESIDENT[name] + NO_ATOMIC_OPT
    cmd = [HIPCC, *FLAGS, *more, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=16) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
