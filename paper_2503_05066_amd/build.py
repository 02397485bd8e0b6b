"""Build libcapmoe.so (the HIP kernels and their C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
if not __package__:  # run as a file
    sys.path.insert(0, os.path.dirname(PKG))
from paper_2503_05066_amd import accumulators  # noqa: E402

ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libcapmoe.so")

SOURCES = ["api.hip", "route.hip", "router_mfma.hip", "drop.hip", "permute.hip", "ffn.hip", "ffn_f32.hip", "ffn_thin.hip", "probe.hip"]
# the packed-fp32 feature is switched off for all device code; the first sixteen words of a kernel's arguments arrive in
# registers (a token through 64 experts x 2048 x 1024: 38.3 -> 37.7 us); the router file must not contract
# multiplies and adds (its softmax is a fixed sequence of individually rounded operations)
COMMON = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-mllvm", "-amdgpu-kernarg-preload-count=16", "-Wall",
          "-Wno-unused-command-line-argument"]
PER_FILE = {"route.hip": ["-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt"]}
# sources whose asm statements name accumulation registers: the assembly of the same compilation is checked
NAMED_ACCUMULATORS = {"ffn.hip"}


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def compile_source(source: str, obj: str, flags=(), named_accumulators: bool = False, verbose: bool = False) -> None:
    with tempfile.TemporaryDirectory(prefix="capmoe_") as tmp:
        # the intermediate files of a compilation lie beside its object
        out = os.path.join(tmp, os.path.basename(obj)) if named_accumulators else obj
        cmd = [_hipcc(), *COMMON, *flags, *(["-save-temps=obj"] if named_accumulators else []), "-c", source, "-o", out]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0 or verbose:
            sys.stderr.write(r.stdout + r.stderr)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed on " + os.path.basename(source))
        if named_accumulators:
            written, = glob.glob(os.path.join(tmp, "*amdgcn*gfx950*.s"))
            with open(written) as f:
                accumulators.check(f.read())
            shutil.move(out, obj)


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(OBJ, src.replace(".hip", ".o"))
        compile_source(os.path.join(CSRC, src), obj, PER_FILE.get(src, []), src in NAMED_ACCUMULATORS, verbose)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    r = subprocess.run([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link failed")
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
