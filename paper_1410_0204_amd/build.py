"""Builds libtmm.so (HIP, gfx950) in-tree next to this file."""

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libtmm.so")
UNITS = ("tmm.hip", "tmm_bins_1.hip", "tmm_bins_2.hip", "tmm_bins_3.hip")
PARTS = ("tmm_rules.hpp", "tmm_device.hpp", "tmm_persistent.hpp", "tmm_bins.hpp", "tmm_substep.hpp", "tmm_probe.hpp")
SOURCES = [os.path.join(HERE, "csrc", f) for f in UNITS]
HEADERS = [os.path.join(HERE, "csrc", f) for f in PARTS] + [os.path.join(ROOT, "include", "tmm.h")]


def source_hash():
    """Hash of the HIP sources the library is built from (keys measured kernel data to a build)."""
    import hashlib
    h = hashlib.sha256()
    for f in PARTS + UNITS:
        with open(os.path.join(HERE, "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def command(src, out):
    return [
        "hipcc", "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-c",
        "-Wall", "-Wno-unused-result",
        # packed float32 instructions stay disabled for all device code
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
        "-o", out, src,
    ]


def build(verbose: bool = False) -> str:
    """Compiles the translation units side by side and links them."""
    tmp = LIB + ".tmp"
    with tempfile.TemporaryDirectory(prefix="tmm_build_") as d:
        objs = [os.path.join(d, os.path.basename(s) + ".o") for s in SOURCES]
        cmds = [command(s, o) for s, o in zip(SOURCES, objs)]
        if verbose:
            for c in cmds:
                print(" ".join(c), flush=True)
        with ThreadPoolExecutor(max_workers=len(cmds)) as pool:
            list(pool.map(lambda c: subprocess.run(c, check=True), cmds))
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
