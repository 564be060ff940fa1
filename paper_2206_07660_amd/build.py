"""Compile libgw.so (HIP kernels + C ABI + host grids) for gfx950, in-tree."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgw.so")
SOURCES = ["gw_kernels.hip", "gw_sandwich.hip", "gw_polar.hip", "gw_dyson.hip", "gw_wlu.hip", "gw_api.hip", "grids.cpp", "ir.cpp"]


def source_hash():
    """sha256 of the kernel and ABI sources (names counter summaries to a build)."""
    import hashlib
    h = hashlib.sha256()
    for f in ("gw_kernels.hip", "gw_sandwich.hip", "gw_polar.hip", "gw_dyson.hip",
              "gw_wlu.hip", "gw_kernels.h", "gw_device.h", "gw_extents.h", "gw_mu.h", "gw_api.hip"):
        with open(os.path.join(CSRC, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def hipcc():
    for p in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if p and os.path.exists(p):
            return p
    raise RuntimeError("hipcc not found")


def build(verbose=False, arch="gfx950"):
    out_tmp = LIB + ".tmp"
    flags = [f"--offload-arch={arch}", "-O3", "-std=c++17", "-fPIC",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             # MFMA accumulators in arch VGPRs: avoids per-iteration AGPR copies
             "-mllvm", "-amdgpu-mfma-vgpr-form",
             "-Wno-unused-result", "-I", os.path.join(HERE, "..", "include")]
    with tempfile.TemporaryDirectory() as tmp:
        # one compiler process per source, side by side
        objs = [os.path.join(tmp, f + ".o") for f in SOURCES]
        procs = [subprocess.Popen([hipcc(), *flags, "-c", os.path.join(CSRC, f), "-o", o], stdout=subprocess.PIPE,
                                  stderr=subprocess.STDOUT, text=True) for f, o in zip(SOURCES, objs)]
        out = [p.communicate()[0] for p in procs]
        failed = any(p.returncode for p in procs)
        if not failed:
            r = subprocess.run([hipcc(), f"--offload-arch={arch}", "-fPIC", "-shared", "-o", out_tmp] + objs,
                               capture_output=True, text=True)
            out.append(r.stdout + r.stderr)
            failed = r.returncode != 0
    msg = "\n".join(l for l in "".join(out).splitlines() if "packed-fp32-ops" not in l)
    if failed:
        raise RuntimeError("hipcc failed:\n" + msg)
    if verbose and msg.strip():
        print(msg, file=sys.stderr)
    os.replace(out_tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
