"""Builds libvenom.so (HIP, gfx950) in-tree next to this file.  `python -m paper_2310_02065_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libvenom.so")
SOURCES = ["venom_api.hip", "venom_format.hip", "venom_prune.hip", "venom_spmm.hip", "venom_skinny.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed-fp32 instructions are not to be generated on this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    return "hipcc"


def build(verbose: bool = True, extra_flags=()) -> str:
    """Compiles the sources side by side (the product kernel's many variants take minutes by themselves) and links them."""
    flags = [f for f in HIPCC_FLAGS if f != "-shared"]
    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, s + ".o") for s in SOURCES]
        cmds = [[hipcc(), *flags, *extra_flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-c", os.path.join(CSRC, s), "-o", o]
                for s, o in zip(SOURCES, objects)]
        link = [hipcc(), "--offload-arch=gfx950", "-fPIC", "-shared", *objects, "-o", LIB]
        if verbose:
            for cmd in cmds:
                print(" ".join(cmd), flush=True)
        _finish([_start(cmd) for cmd in cmds], verbose)
        _finish([_start(link)], verbose)
    return LIB


def _start(cmd):
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def _finish(running, verbose):
    results = [(p.communicate()[0], p.returncode) for p in running]   # all of them end before one is reported
    for text, code in results:
        out = "\n".join(l for l in text.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if code != 0:
            raise RuntimeError(f"hipcc failed ({code}):\n{out}")
        if verbose and out:
            print(out, flush=True)


if __name__ == "__main__":
    build(extra_flags=sys.argv[1:])
    print("built", LIB)
