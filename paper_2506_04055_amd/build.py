"""Build libmlp.so in-tree for gfx950 with hipcc.

Every HIP source is compiled with packed-FP32 instructions disabled
(``-Xclang -target-feature -Xclang -packed-fp32-ops``).
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libmlp.so")
BUILD = os.path.join(HERE, "_build")
PROBE = os.path.join(os.path.dirname(HERE), "tests", "device", "libprobe.so")
SOURCES = ["api.hip", "nbr.hip", "painn.hip", "prof.hip", "node_p2.hip", "node_p0.hip", "node_p1.hip", "gemm.hip", "node.hip", "msg.hip", "server.hip", "md.hip", "noalloc.hip", "allegro.hip",
           "mace.hip"]
ARCH = os.environ.get("MLP_OFFLOAD_ARCH", "gfx950")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result", "-Wno-unused-command-line-argument",
]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *CFLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed on {src}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(4, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link of libmlp.so failed")
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


def build_probe() -> str:
    """The tests' device probe (tests/device/probe.hip) as a library of its own, with the same flags."""
    tmp = PROBE + ".tmp"
    r = subprocess.run([HIPCC, *CFLAGS, "-shared", os.path.join(os.path.dirname(PROBE), "probe.hip"), "-o", tmp],
                       capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed on probe.hip")
    os.replace(tmp, PROBE)
    return PROBE


def probe_lib() -> str:
    """The built probe; built first where there is none."""
    return PROBE if os.path.exists(PROBE) else build_probe()


if __name__ == "__main__":
    build(verbose=True)
