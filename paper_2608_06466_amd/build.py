"""Build libzoneburn.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2608_06466_amd.build [--jobs N] [--verbose]
"""
import argparse
import hashlib
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libzoneburn.so")
# the burn-kernel instantiations are spread over several files so they compile in parallel
SOURCES = [
    # the 48-row kernels compile slowest: first, so the parallel build starts them early
    "zb_k48d.hip", "zb_k48f.hip", "zb_k48dr.hip", "zb_k48fr.hip",
    "zb_kv_d.hip", "zb_kv_e.hip", "zb_kvr_d.hip", "zb_kvr_e.hip", "zb_k48b.hip",
    "zb_k16.hip", "zb_k14.hip", "zb_k14r.hip", "zb_k14v.hip", "zb_k14vr.hip", "zb_k22.hip",
    "zb_k22r.hip", "zb_k16r.hip", "zb_k16n.hip", "zb_k24.hip", "zb_k24r.hip", "zb_k32.hip",
    "zb_k32r.hip", "zb_k04.hip", "zb_k04r.hip", "zb_kc.hip",
    "zb_kv_a.hip", "zb_kv_b.hip", "zb_kv_c.hip", "zb_kvr_a.hip", "zb_kvr_b.hip", "zb_kvr_c.hip",
    "zb_kernels.hip", "zb_host.hip", "zb_server.hip",
]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed FP32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # keep hoisted FP64 constants from flooding the scalar registers of the large kernels
    "-mllvm", "-disable-machine-licm",
    "-Wall", "-Wno-unused-function", "-Wno-unused-variable",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# Machine-scheduler strategy per kernel class, as measured: the 16-, 22-, 24- and 32-row kernels
# run 1-3 % faster with max-ilp, the 48-row ones 5-9 % faster with iterative-ilp; the small
# kernels keep the default, and so do the 14-row ones but for their variable form without reuse.
# Default and max-ilp on 14 variables, 100003 zones: reuse mixed 166 and 174 ms, FP64 189.1 and
# 190.2; variable form with reuse mixed 210 and 218, FP64 223 and 225; without reuse mixed 237.4
# and 238.6, FP64 239.3 and 236.8; every step, 2^18 zones mixed 428 and 437, 50021 zones FP64 97.4
# and 99.0.
SCHED = {
    **{f: "max-ilp" for f in ("zb_k16.hip", "zb_k14v.hip", "zb_k22.hip", "zb_k22r.hip", "zb_k16r.hip", "zb_k16n.hip", "zb_k24.hip",
                              "zb_k24r.hip", "zb_k32.hip", "zb_k32r.hip", "zb_kv_b.hip",
                              "zb_kv_c.hip", "zb_kvr_b.hip", "zb_kvr_c.hip")},
    **{f: "iterative-ilp" for f in ("zb_k48d.hip", "zb_k48f.hip", "zb_k48dr.hip", "zb_k48fr.hip",
                                    "zb_kv_d.hip", "zb_kv_e.hip", "zb_kvr_d.hip", "zb_kvr_e.hip",
                                    "zb_k48b.hip")},
}


def kernels_id():
    """Identifies the burn kernels of a build (their sources, flags and scheduling): saved tuning
    files carry it, since other kernels have other fastest mappings."""
    h = hashlib.sha256(repr(([f for f in FLAGS if not os.path.isabs(f)], sorted(SCHED.items()))).encode())
    for f in sorted(os.listdir(CSRC)):
        if f.startswith("zb_k") and f.endswith(".hip") or f in (
                "zb_burn_kernel.h", "zb_internal.h", "zb_log.h", "zb_stepmath.h"):
            with open(os.path.join(CSRC, f), "rb") as s:
                h.update(s.read())
    return h.hexdigest()[:16]


def _compile(src, verbose):
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    extra = ["-mllvm", f"-amdgpu-sched-strategy={SCHED[src]}"] if src in SCHED else []
    if src == "zb_host.hip":
        extra.append(f'-DZB_KERNELS_ID="{kernels_id()}"')
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return obj


def build(jobs=None, verbose=False):
    os.makedirs(OBJ, exist_ok=True)
    jobs = jobs or min(len(SOURCES), os.cpu_count() or 1)
    with ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    ap.add_argument("--jobs", type=int, default=None)
    ap.add_argument("--verbose", action="store_true")
    a = ap.parse_args()
    build(a.jobs, a.verbose)
    sys.exit(0)
