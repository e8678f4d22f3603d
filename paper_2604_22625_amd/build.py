"""Build the HIP library libffolio.so in-tree for gfx950 (and the C oracle checks, if any).

Usage: python -m paper_2604_22625_amd.build   (or call build() from Python).
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libffolio.so")
SOURCES = ["ffolio_host.hip", "solve_kernel.hip", "reg_kernel.hip", "mp_kernel.hip", "setup_kernels.hip", "lockstep.hip", "riskmodel.hip"]
ARCH = os.environ.get("FFO_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (set HIPCC)")


def flags() -> list[str]:
    return [f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
            # packed FP32 instructions stay off for every kernel of this library
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include")]


def build(verbose: bool = False) -> str:
    tmp = LIB + ".tmp"
    # a failed build must not leave an older library behind to be loaded by mistake
    if os.path.exists(LIB):
        os.remove(LIB)
    with tempfile.TemporaryDirectory() as objs:
        out = [os.path.join(objs, s + ".o") for s in SOURCES]
        # one compiler per source, all at once: the templates of three sources take minutes each
        with ThreadPoolExecutor(min(len(SOURCES), os.cpu_count() or 1)) as pool:
            list(pool.map(lambda so: _run([hipcc()] + flags() + ["-c", os.path.join(CSRC, so[0]), "-o", so[1]], verbose),
                          zip(SOURCES, out)))
        _run([hipcc(), f"--offload-arch={ARCH}", "-fPIC", "-shared", "-o", tmp] + out, verbose)
    os.replace(tmp, LIB)
    return LIB


def _run(cmd, verbose) -> None:
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
