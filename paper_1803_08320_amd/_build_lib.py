"""Build libmalbec.so (HIP, gfx950) in-tree with hipcc.

Every translation unit under csrc/ is compiled to an object in _build/ and the
objects are linked into paper_1803_08320_amd/libmalbec.so.  All HIP code is
compiled with packed-FP32 instruction selection disabled.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmalbec.so")
ARCH = os.environ.get("MALBEC_OFFLOAD_ARCH", "gfx950")

COMMON = ["-O3", "-std=c++17", "-fPIC", "-ffp-contract=on", "--offload-arch=" + ARCH,
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-fvisibility=hidden", "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument"]

# These kernels are chains of dependent arithmetic at one to four waves per SIMD: scheduled
# for instruction-level parallelism rather than for occupancy, and not reordered again after
# register allocation.  On one MI355X against the default (the same results): 1,024 Kerr lanes
# x 1,000 steps 0.867 -> 0.850 ms, in the Hamiltonian form 0.739 -> 0.707, 262,144 lanes 3.02 ->
# 2.99 and 2.42 -> 2.39 ms, 20,000 monitored lanes 0.920 -> 0.896 ms, the gridded kernel (262,144
# lanes x 400 steps) 6.42 -> 6.10 ms, a 512 x 512 camera image 3.14 -> 3.03 ms, 262,144
# FP32-compensated lanes x 600 steps 1.33 -> 1.25 ms.  The adaptive kernel is slower with it
# (262,144 lanes 4.95 -> 5.14 ms), and it changes nothing for the adjoint.  The monitored
# FP32-compensated queue of the Hamiltonian form takes 3 to 5 % more with it at 230,000 to 262,144
# lanes, and up to 3 % less from 400,000 on.
SCHEDULE = ["-mllvm", "-amdgpu-sched-strategy=max-ilp", "-mllvm", "-enable-post-misched=0"]
SCHEDULED = ("camera.hip", "grid.hip", "integrate.hip", "mixed.hip", "trajectory.hip")


def hipcc() -> str:
    for cand in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"),
                 shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP toolchain is required to build libmalbec")


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, src[:-4] + ".o")
    cmd = [hipcc()] + COMMON + (SCHEDULE if src in SCHEDULED else []) + ["-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, " ".join(cmd), res.stderr))
    return obj


def build(jobs: int = 8) -> str:
    """Compile every csrc/*.hip and link libmalbec.so; returns the library path."""
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=max(1, min(jobs, 16))) as ex:
        objs = list(ex.map(_compile, sources()))
    tmp = LIB + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp] + objs
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (" ".join(cmd), res.stderr))
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
