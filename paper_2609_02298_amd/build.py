"""Build the gfx950 HIP library ``libib_lbm.so`` in-tree with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libib_lbm.so")
SOURCES = ["lbm_kernels.hip", "ibm_kernels.hip", "step_kernels.hip", "measure_kernels.hip", "host_copy.cpp", "ib_lbm_api.cpp",
           "ib_lbm_server.cpp"]
ARCH = os.environ.get("IB_LBM_ARCH", "gfx950")
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
         # packed FP32 instructions are kept out of the generated code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]
# The collide-stream kernels write every fused multiply-add out explicitly,
# so that all their instances round alike: no automatic contraction there.
# The IB pass contracts within an expression only: its instances (separate
# launch, one-launch step) then round alike, whatever code surrounds them.
PER_SOURCE = {"lbm_kernels.hip": ["-ffp-contract=off"], "ibm_kernels.hip": ["-ffp-contract=on"],
              "step_kernels.hip": ["-ffp-contract=on"]}


def _compile(src: str) -> tuple[str, str]:
    obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".cpp") else []
    cmd = ["hipcc", *FLAGS, *PER_SOURCE.get(src, []), *lang, "-c", os.path.join(CSRC, src),
           "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    msg = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{msg}")
    return obj, msg


def build(verbose: bool = False) -> str:
    objs = []
    with ThreadPoolExecutor(4) as ex:
        for obj, msg in ex.map(_compile, SOURCES):
            if verbose and msg.strip():
                print(msg, file=sys.stderr)
            objs.append(obj)
    tmp = LIB + ".tmp"
    cmd = ["hipcc", f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, LIB)
    for o in objs:
        os.remove(o)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
