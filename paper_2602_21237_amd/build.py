"""Builds libtj.so (HIP kernels + C-ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import concurrent.futures
import glob
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIBDIR = os.path.join(HERE, "lib")
LIB = os.path.join(LIBDIR, "libtj.so")
SOURCES = ["tj_kernels.hip", "tj_rmi.hip", "tj_multi.hip", "tj_abi.cpp", "tj_serve.cpp", "tj_multi.cpp", "tj_static.hip", "tj_fuse.hip", "tj_bandwidth.hip",
           "tj_select.hip", "tj_select.cpp"]
HEADERS = ["tj_internal.h", "tj_events.h", "tj_rmi.h", "tj_select.h"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Packed FP32 instructions are disabled for all device code; the host pass
# ignores the feature (and warns).
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


_FUNCTION = re.compile(r"^([A-Za-z_]\w*):")
_BLOCK = re.compile(r"^(\.LBB\S*:|; %bb\.)")
_SPILL = re.compile(r"\s(scratch_store\S*|buffer_store\S*|v_accvgpr_write\S*)\s.*Folded Spill")
_LANES_BACK = re.compile(r"\ss_or_b64 exec, exec,")


def lost_lanes(listing: str) -> list:
    """Spills of vector registers, in the assembly of a device build, that stand
    ahead of the instruction that gives their block its lanes back: the lanes
    that come back have stored nothing, and read another value when the register
    is reloaded. (The compiler has placed some so at the end of loops, in blocks
    that have every register in use; results were wrong with no error.)
    Returns "function: instruction" for each."""
    bad, pending, function = [], [], "?"
    for line in listing.splitlines():
        m = _FUNCTION.match(line)
        if m and not line.startswith(".L"):
            function, pending = m.group(1), []
        elif _BLOCK.match(line):
            pending = []
        elif _SPILL.search(line):
            pending.append("%s: %s" % (function, line.strip()))
        elif _LANES_BACK.search(line):
            bad += pending
            pending = []
    return bad


def build(verbose: bool = False) -> str:
    """Compiles every HIP/C++ source of the library into lib/libtj.so. Fails where
    the compiler has spilled registers of lanes that it then loses (lost_lanes)."""
    os.makedirs(LIBDIR, exist_ok=True)
    with tempfile.TemporaryDirectory() as tmp:
        def compile_one(source: str) -> str:
            at = os.path.join(tmp, source)  # a folder of its own: the listings are named without the suffix
            os.mkdir(at)
            obj = os.path.join(at, source + ".o")
            cmd = [HIPCC, "-x", "hip"] + FLAGS + ["-I", os.path.join(ROOT, "include"), "-save-temps=obj", "-c",
                                                  os.path.join(CSRC, source), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            run = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            if verbose or run.returncode:
                print(run.stdout, flush=True)
            run.check_returncode()
            return obj

        with concurrent.futures.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            objs = list(pool.map(compile_one, SOURCES))
        listings = glob.glob(os.path.join(tmp, "*", "*gfx950*.s"))
        if len(listings) != len(SOURCES):
            raise RuntimeError("device listings of %d of %d sources" % (len(listings), len(SOURCES)))
        for path in sorted(listings):
            with open(path) as f:
                bad = lost_lanes(f.read())
            if bad:
                raise RuntimeError("%s: spills before their lanes are back:\n%s" % (os.path.basename(path), "\n".join(bad)))
        lib = LIB + ".tmp%d" % os.getpid()
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", lib] + objs)
        os.replace(lib, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
