"""Build libgreencache.so (the HIP kernels and the C ABI) for gfx950 with hipcc,
and libgreencache_ctl.so (the CPU replacement model) with g++.

Run as `python -m paper_2505_23970_amd.build`; writes the libraries next to
this file so that they travel with the source tree.
"""
from __future__ import annotations

import concurrent.futures
import glob
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBRARY = os.path.join(HERE, "libgreencache.so")
ARCH = "gfx950"

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-fvisibility=hidden", "-Wall",
    # keep the compiler from forming packed fp32 arithmetic
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

CONTROL_LIBRARY = os.path.join(HERE, "libgreencache_ctl.so")
# IEEE double without contraction: the replacement scores are compared exactly
CONTROL_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-ffp-contract=off",
                 "-Wall", "-Wextra"]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def build_control(out: str = CONTROL_LIBRARY) -> str:
    tmp = out + f".tmp{os.getpid()}"
    cmd = ["g++", *CONTROL_FLAGS, "-I", os.path.join(ROOT, "include"),
           os.path.join(CSRC, "cache_policy.cpp"), "-o", tmp]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed ({res.returncode}):\n{res.stdout}")
    os.replace(tmp, out)
    return out


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 feature and says so; drop that noise
    noise = "is not a recognized feature for this target"
    msg = "\n".join(l for l in res.stdout.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed ({res.returncode}):\n{msg}")
    if msg.strip() and verbose:
        print(msg)


def build(out: str = LIBRARY, extra=(), verbose=False) -> str:
    """Compile every source to an object (in parallel), then
    link the shared library; always from scratch."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = out + f".tmp{os.getpid()}"
    with tempfile.TemporaryDirectory(prefix="gc_build_") as objdir:
        jobs = []
        for src in sources():
            obj = os.path.join(objdir, os.path.basename(src) + ".o")
            jobs.append(([hipcc, *HIPCC_FLAGS, *extra,
                          "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", src, "-o", obj], obj))
        workers = max(1, min(len(jobs), os.cpu_count() or 1, 8))
        with concurrent.futures.ThreadPoolExecutor(workers) as pool:
            for f in [pool.submit(_run, cmd, verbose) for cmd, _ in jobs]:
                f.result()
        _run([hipcc, "-shared", "-fPIC", f"--offload-arch={ARCH}", *[o for _, o in jobs], "-o", tmp], verbose)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
    print(build_control())
