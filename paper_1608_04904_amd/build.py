"""Compile librmpmd.so for gfx950 with hipcc (in-tree): one object per source,
compiled in parallel, then linked."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = [os.path.join(HERE, "csrc", f) for f in ("rmp_capi.hip", "rmp_chain_f64.hip", "rmp_chain_f32.hip")]
OUT = os.path.join(HERE, "librmpmd.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # every floating-point operation rounds separately unless written as fma()
    "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + r.stderr[-4000:])

    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SRC]
        with ThreadPoolExecutor(len(SRC)) as ex:
            list(ex.map(run, ([hipcc, *HIPCC_FLAGS, "-c", s, "-o", o] for s, o in zip(SRC, objs))))
        run([hipcc, "--offload-arch=gfx950", "-fPIC", "-shared", *objs, "-o", OUT + ".tmp"])
    os.replace(OUT + ".tmp", OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose=True))
