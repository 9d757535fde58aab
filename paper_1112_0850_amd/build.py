"""Build the gfx950 HIP library ``liblbm.so`` in-tree with hipcc.

Every call compiles from source.  Flags: gfx950 only, -O3, and packed-FP32
instructions disabled (-packed-fp32-ops) for all device code.
"""
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblbm.so")
# (source, defines) of each object; kernels.hip is compiled in parts
SOURCES = [("kernels.hip", [f"-DLBM_PART={p}"]) for p in range(11)] + [("abi.hip", [])]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# -ffp-contract=on: multiply-adds are fused only inside one source
# expression, as written, so every template instantiation of the collision
# (wall kinds, split or fused bounce-back, cells per lane) rounds identically;
# the default cross-statement fusion pairs products differently per kernel.
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=on",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fvisibility=hidden", "-Wall", "-Wno-unused-result",
    "-I" + os.path.join(ROOT, "include"),
]


def build(verbose: bool = False, extra=()) -> str:
    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    flags = [f for f in FLAGS if f != "-shared"] + list(extra)
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(8) as pool:
        objs = [os.path.join(tmp, f"{k}.o") for k in range(len(SOURCES))]
        list(pool.map(run, [[HIPCC] + flags + defs + ["-c", os.path.join(CSRC, src), "-o", obj]
                            for (src, defs), obj in zip(SOURCES, objs)]))
        run([HIPCC] + FLAGS + objs + ["-o", LIB + ".tmp"])
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
