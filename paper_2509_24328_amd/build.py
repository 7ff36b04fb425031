"""Build the HIP library for gfx950 in-tree: paper_2509_24328_amd/libsv.so."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libsv.so")
SOURCES = ["row_stats.hip", "warp.hip", "verify_sample.hip", "select_length.hip", "profile.hip", "sparse.hip",
           "accept_estimate.hip", "penalty.hip", "api.hip"]
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-shared",
         # products are fused only where the code says fmaf: the online
         # accumulator relies on c(m) being the same rounded fp32 number
         # everywhere it is used
         "-ffp-contract=off",
         # packed-fp32 code generation is switched off on this target
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
OWN_FLAGS = {
    # the constants of an fp64 logarithm or exponential stay where they are used: hoisted out of the loop
    # over pairs they take dozens of the registers that hold the rows.  (Not for the others: the sweeps of
    # deep nuclei in warp.hip are 2 % slower with it.)
    "row_stats.hip": ["-mllvm", "-disable-machine-licm"],
}


def build(verbose=False):
    """Compile every HIP source, side by side, and link libsv.so (always recompiles)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)

    with tempfile.TemporaryDirectory() as tmp:
        objects = [os.path.join(tmp, s + ".o") for s in SOURCES]
        flags = [f for f in FLAGS if f != "-shared"]
        cmds = [[hipcc] + flags + OWN_FLAGS.get(s, []) + ["-c", os.path.join(CSRC, s), "-o", o]
                for s, o in zip(SOURCES, objects)]
        with ThreadPoolExecutor(max_workers=4) as pool:
            list(pool.map(run, cmds))
        run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objects)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
