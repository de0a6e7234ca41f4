"""Build of the HIP library ``liblbm_cde.so`` for gfx950 (in-tree).

The library is compiled from the ``csrc/*.hip`` sources with hipcc, one
process per source (each holds kernels of its own), and linked.  Packed FP32
instructions are disabled for the device code.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "liblbm_cde.so")
SOURCES = [os.path.join(HERE, "csrc", f) for f in
           ("lbm_cde.hip", "box_f32.hip", "box_f64.hip", "small_f32.hip", "small_f64.hip", "strip_f32.hip",
            "strip_f64.hip", "vol.hip")]
ARCH = os.environ.get("LBM_CDE_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP library cannot be built")


def command(src: str, out: str) -> list:
    return [hipcc(), "-O3", "-std=c++17", f"--offload-arch={ARCH}", "-fPIC", "-c", "-ffp-contract=on",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
            "-o", out, src]


def build(verbose: bool = False) -> str:
    """Compile the library (always) and return its path."""
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, os.path.basename(src) + ".o") for src in SOURCES]
        steps = [command(src, obj) for src, obj in zip(SOURCES, objects)]
        link = [hipcc(), f"--offload-arch={ARCH}", "-fPIC", "-shared", "-o", LIB + ".tmp"] + objects
        if verbose:
            for cmd in steps + [link]:
                print(" ".join(cmd), flush=True)
        logs = [open(obj + ".log", "w+") for obj in objects]
        procs = [subprocess.Popen(cmd, stdout=log, stderr=subprocess.STDOUT) for cmd, log in zip(steps, logs)]
        failed = any([p.wait() for p in procs])
        for log in logs:
            log.seek(0)
            if failed:
                sys.stderr.write(log.read())
            log.close()
        if failed:
            raise RuntimeError("hipcc failed building liblbm_cde.so")
        res = subprocess.run(link, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError("hipcc failed linking liblbm_cde.so")
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
