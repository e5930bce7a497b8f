"""Build librc.so (HIP for gfx950) in-tree.

Every translation unit is compiled with -ffp-contract=off (the LUT entry is a
fixed, uncontracted binary64 sequence) and without packed FP32 instructions.
"""
import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJ = os.path.join(ROOT, "_build", "rc")
LIB = os.path.join(PKG, "librc.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

FLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-fno-fast-math", "-Wall", "-Wno-unused-result",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", INCLUDE, "-I", CSRC]
# lut_apply.hip holds 240 correction kernels: each (pixels per lane, lines per
# register set) is compiled as its own unit, in parallel (one unit took 4
# minutes).
APPLY_SHAPES = [(8, 4), (4, 16), (4, 8), (2, 16), (4, 4), (2, 8), (1, 16), (2, 4), (1, 8), (1, 4)]
SOURCES = ["lut_build.hip", "lut_apply.hip", "batch.hip", "fit.hip", "demosaic.hip",
           "demosaic_gradient.hip", "stream_copy.hip", "noalloc.hip", "api.cpp", "tune.cpp",
           "serve.cpp", "wire.cpp"]


def _units():
    """(source, defines, object) of every translation unit, the longest first."""
    units = [("lut_apply.hip", [f"-DRC_APPLY_VEC={v}", f"-DRC_APPLY_UNROLL={u}"],
              f"lut_apply_{v}_{u}.o") for v, u in APPLY_SHAPES]
    return units + [(src, [], os.path.basename(src) + ".o") for src in SOURCES]


def _compile(unit):
    src, defines, obj = unit
    out = os.path.join(OBJ, obj)
    cmd = [HIPCC, *FLAGS, *defines, "-c", os.path.join(CSRC, src), "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")
    return out


def build(quiet=True):
    os.makedirs(OBJ, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(_compile, _units()))
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", *objs, "-o", LIB + ".tmp",
           "-lpthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{res.stderr}")
    os.replace(LIB + ".tmp", LIB)
    if not quiet:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(quiet=False)
    sys.exit(0)
