"""Compile the HIP sources under csrc/ into paper_2604_04701_amd/libmuxq.so (gfx950)."""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmuxq.so")
SOURCES = ["muxq_api.hip", "muxq_scan.hip", "muxq_gemm.hip", "muxq_gemm_own.hip",
           "muxq_gemm_gelu.hip", "muxq_gemm_codes.hip", "muxq_few.hip", "muxq_act.hip", "muxq_probe.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "--offload-arch=gfx950"
FLAGS = [
    ARCH, "-O3", "-std=c++17", "-fPIC",
    "-ffp-contract=off",                      # the fp32 op order of the scales is part of the contract
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False, extra=()) -> str:
    """One compiler per source, several at a time, then the link."""
    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        msgs = "\n".join(l for l in (res.stdout + res.stderr).splitlines()
                         if "packed-fp32-ops" not in l and l.strip())
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + msgs)
        if verbose and msgs:
            print(msgs)

    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, s.replace(".hip", ".o")) for s in SOURCES]
        with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            list(pool.map(run, [[HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, s), "-o", o]
                                for s, o in zip(SOURCES, objs)]))
        run([HIPCC, ARCH, "-fPIC", "-shared", *objs, "-o", LIB])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
