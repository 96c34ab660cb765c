"""Builds libvarco.so (HIP kernels + C ABI, gfx950 only) next to this file with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libvarco.so")
SOURCES = ["varco_api.hip", "varco_network.hip", "kernels_network.hip", "kernels_compress.hip", "kernels_spmm.hip", "kernels_gemm.hip", "kernels_gemm_bf16.hip", "kernels_gemm_tn_bf16.hip", "kernels_gemm_rows.hip", "kernels_gemm_split.hip", "kernels_gemm_split_rows.hip", "kernels_gemm_half.hip", "kernels_gemm_half_tn.hip", "kernels_gemm_half_nt.hip", "kernels_halo_transform.hip", "kernels_class_first.hip", "kernels_train.hip", "partition_builder.cpp"]
# -packed-fp32-ops is switched off for every device compilation of this library (packed fp32 forms have
# produced wrong values on the target boxes); the host pass does not know the feature and says so.
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def build(verbose: bool = False) -> str:
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = []
    procs = []
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        objs.append(obj)
        cmd = [hipcc, *FLAGS, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        lines = [l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip()]
        if p.returncode != 0:
            failed = True
            print(f"--- {src} failed ---\n" + "\n".join(lines), file=sys.stderr)
        elif verbose and lines:
            print(f"--- {src} ---\n" + "\n".join(lines))
    if failed:
        raise RuntimeError("hipcc failed")
    cmd = [hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", *objs, "-o", LIB]
    subprocess.run(cmd, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
