"""Build the HIP library ``liblbm_hip.so`` for gfx950 (in-tree).

    python -m paper_2309_02825_amd.build

The kernel sources are compiled side by side and linked.  Every HIP source is
compiled with packed-FP32 instructions disabled (the kernels are FP64; this
keeps the compiler from emitting packed FP32 forms in any float code).
"""
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "liblbm_hip.so")
# the slowest to compile first
SOURCES = [os.path.join(CSRC, n) for n in
           ("lbm_d2q9_s8_mom.hip", "lbm_d2q9_s8_full.hip", "lbm_d2q9_s8_twin.hip",
            "lbm_batch.hip", "lbm_d2q9_adjoint.hip", "lbm_d2q9_s4.hip",
            "lbm_d2q9_s2.hip", "lbm_d2q9_tile.hip", "lbm_d3q19.hip",
            "lbm_d3q19_march.hip", "lbm_kernels.hip", "lbm_d1.hip", "lbm_api.hip",
            "lbm_d2q9.hip")]
ARCH = os.environ.get("LBM_OFFLOAD_ARCH", "gfx950")


def hipcc_flags():
    # no floating-point contraction: every kernel that runs the same
    # collision performs the same roundings (fused multi-step passes and the
    # batched form are bitwise equal to single steps)
    return ["-O3", "-ffp-contract=off", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument",
            "-I", INCLUDE, "-I", CSRC]


def build(verbose: bool = False) -> str:
    def compile_one(job):
        src, obj = job
        cmd = ["hipcc"] + hipcc_flags() + ["-c", "-o", obj, src]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)

    with tempfile.TemporaryDirectory() as objdir:
        jobs = [(s, os.path.join(objdir, os.path.basename(s) + ".o")) for s in SOURCES]
        workers = max(1, min(len(jobs), int(os.environ.get("MAX_JOBS", os.cpu_count() or 1))))
        with ThreadPoolExecutor(workers) as pool:
            list(pool.map(compile_one, jobs))
        tmp = LIB + ".tmp"
        cmd = ["hipcc", f"--offload-arch={ARCH}", "-fPIC", "-shared", "-o", tmp] + [o for _, o in jobs]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
