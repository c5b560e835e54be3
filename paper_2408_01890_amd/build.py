"""Compile the HIP sources into ``liblisa_mi355x.so`` inside the package (gfx950 only)."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblisa_mi355x.so")
# (source, parts): a source with many kernel instantiations is compiled in parts, side by side, each with
# -DLISA_PART=<its number>
UNITS = [("launch_prefill.hip", 5), ("launch_decode.hip", 1), ("launch_stack.hip", 1), ("launch_f32.hip", 1), ("launch_split.hip", 1),
         ("launch_scores.hip", 1), ("lisa_api.hip", 1)]
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory(prefix="lisa_build_") as tmp:
        objs, cmds = [], []
        for src, parts in UNITS:
            for part in range(parts):
                objs.append(os.path.join(tmp, f"{src}.{part}.o"))
                cmds.append([hipcc, *FLAGS, f"-DLISA_PART={part}", "-c", "-o", objs[-1], os.path.join(CSRC, src)])

        def run(cmd):
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)

        with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            list(pool.map(run, cmds))
        run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
