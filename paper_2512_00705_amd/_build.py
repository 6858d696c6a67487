"""Build libflexiwalk.so for gfx950 with hipcc (in-tree)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libflexiwalk.so")
SOURCES = ["fw_trial_node2vec.hip", "fw_trial_secondpr.hip", "fw_trial_metapath.hip", "fw_rvs.hip", "fw_kernels.hip",
           "fw_api.hip", "fw_server.hip"]

# -ffp-contract=off: no fused multiply-add anywhere, so float32 results follow the
#   stated operation order; denormals are kept; packed fp32 ops are disabled.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-fno-gpu-flush-denormals-to-zero", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
    # an atomic's result is used a pass later; the optimizer's rewrite would wait for it at once
    "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
]


def build(verbose: bool = False, out: str = LIB, defines=(), objdir: str = CSRC) -> str:
    """Compile every source and link ``out``.  ``defines`` ("NAME=VALUE") set tuning knobs."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(objdir, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        cmd = [hipcc, *FLAGS, *[f"-D{d}" for d in defines], "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = out + ".tmp"
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp, "-lpthread"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, out)
    return out


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
