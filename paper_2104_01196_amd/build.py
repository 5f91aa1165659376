"""Build libgs2.so (the HIP C-ABI library) for gfx950 with hipcc.

Usage: python -m paper_2104_01196_amd.build   (or call build())
Object files go to paper_2104_01196_amd/_build/, the library next to this file.
"""
from __future__ import annotations

import os
import re
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libgs2.so")
SOURCES = ["setup.hip", "sweep.hip", "sella.hip", "krylov.hip", "resident.hip", "small.hip", "cg.hip", "batched.hip", "profile.hip"]
ARCH = os.environ.get("GS2_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-Wall",
    "-Wno-unused-result",
    # packed-FP32 instructions are disabled for the whole library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I", os.path.join(ROOT, "include"),
]


# Kernels that must not spill vector registers or use scratch memory: an
# instantiation of k_resident that spilled 55 vector registers beside 139 scalar
# ones gave wrong results, the same ones every time, and the same source without
# spills right ones.  (Scalar registers alone go to lanes of vector registers.)
NO_SPILLS = {"resident.hip": "k_resident", "small.hip": "k_small_apply"}


def check_spills(remarks: str, kernel: str) -> int:
    """Instantiations of `kernel` in the compiler's resource remarks; raises if one spills."""
    seen = 0
    for block in remarks.split("Function Name: ")[1:]:
        name = block.split()[0]
        if kernel not in name:
            continue
        seen += 1
        for what in ("VGPRs Spill", r"ScratchSize \[bytes/lane\]"):
            m = re.search(what + r": (\d+)", block)
            if m is None or int(m.group(1)) != 0:
                raise RuntimeError(f"{name}: {m.group(0) if m else 'no ' + what} (must be 0)")
    if not seen:
        raise RuntimeError(f"no resource remarks for {kernel}")
    return seen


def _hipcc() -> str:
    h = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(h):
        raise RuntimeError("hipcc not found: the HIP library cannot be built")
    return h


def _runtime_dir() -> str:
    """Directory of the libamdhip64.so the process will use (torch's bundled
    copy when torch is installed, else the ROCm installation)."""
    try:
        import importlib.util

        spec = importlib.util.find_spec("torch")
        if spec and spec.origin:
            d = os.path.join(os.path.dirname(spec.origin), "lib")
            if os.path.exists(os.path.join(d, "libamdhip64.so")):
                return d
    except Exception:
        pass
    return "/opt/rocm/lib"


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    if src in NO_SPILLS:
        cmd.append("-Rpass-analysis=kernel-resource-usage")
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    if src in NO_SPILLS:
        check_spills(r.stderr, NO_SPILLS[src])
    errs = [ln for ln in r.stderr.splitlines() if "warning" in ln and "packed-fp32-ops" not in ln
            and "recognized feature" not in ln]
    if errs:
        sys.stderr.write("\n".join(errs) + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = [s for s in SOURCES if os.path.exists(os.path.join(CSRC, s))]
    with ThreadPoolExecutor(max_workers=min(4, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + f".tmp{os.getpid()}"
    # Link against the HIP runtime that torch loads, so that a process using
    # torch for device memory and streams holds a single HIP runtime.
    rt = _runtime_dir()
    cmd = ["g++", "-shared", "-fPIC", "-o", tmp, *objs, f"-L{rt}", "-l:libamdhip64.so", f"-Wl,-rpath,{rt}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link of libgs2.so failed")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


if __name__ == "__main__":
    build()
