"""Builds libjf.so (HIP, gfx950) in-tree: paper_2512_14681_amd/libjf.so.

    python -m paper_2512_14681_amd.build
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(os.path.dirname(HERE), "_build")
LIB = os.path.join(HERE, "libjf.so")
SOURCES = ["jf_api.hip", "gemm.hip", "gemm_mr.hip", "gemm_mr_any.hip",
           *(f"gemm_mr_rt{n}.hip" for n in (2, 4, 6, 8, 10, 12, 16)), "attention.hip", "layer.hip", "step.hip",
           "trajectory.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17", "-Wall",
         "-Wno-unused-function", "-Wno-unused-variable",
         # no packed fp32 instructions (v_pk_*_f32) in any device code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _run(cmd):
    r = subprocess.run(cmd, capture_output=True, text=True)
    # the host pass does not know the packed-fp32 feature; that warning is noise
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    return r.returncode, err


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    objs = [os.path.join(BUILD, s.replace(".hip", ".o")) for s in SOURCES]
    cmds = [[HIPCC, *FLAGS, "-c", os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objs)]
    with ThreadPoolExecutor(min(8, len(cmds))) as ex:
        results = list(ex.map(_run, cmds))
    for (rc, err), s in zip(results, SOURCES):
        if err.strip() and (verbose or rc):
            print(f"[{s}]\n{err}", file=sys.stderr)
        if rc:
            raise RuntimeError(f"hipcc failed on {s}")
    tmp = LIB + ".tmp"
    rc, err = _run([HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", tmp])
    if rc:
        print(err, file=sys.stderr)
        raise RuntimeError("link failed")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
