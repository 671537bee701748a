"""Builds libozimmu.so (HIP, gfx950) in-tree with hipcc.  No torch extension machinery: the
library has a plain C ABI and is loaded with ctypes."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libozimmu.so")
SOURCES = ["api.hip", "reduce.hip", "split.hip", "gemm.hip", "gemm_fused16.hip", "gemm_banded.hip", "gemm_small.hip", "gemm_vectors.hip",
           "gemm_halves16.hip", "gemm_passes.hip", "gemm_passes_4.hip", "gemm_passes_10.hip", "gemm_passes_13.hip", "gemm_passes_15.hip", "gemm_passes_17.hip", "gemm_passes_19.hip", "ceiling.hip"]
HEADERS = [os.path.join(CSRC, "oz_common.h"), os.path.join(CSRC, "gemm_dev.h"), os.path.join(CSRC, "gemm_passes_dev.h"), os.path.join(CSRC, "slice_dev.h"), os.path.join(HERE, "..", "include", "ozimmu.h"),
           os.path.join(HERE, "..", "include", "ozimmu_bench.h")]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-fast-math", "-ffp-contract=on",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def _stale(target, deps):
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def build_lib(force=False, verbose=False):
    """Compile every HIP source and link the shared library.  Returns its path."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    for src in SOURCES:
        spath = os.path.join(CSRC, src)
        obj = os.path.join(CSRC, src.replace(".hip", ".o"))
        objs.append(obj)
        if force or _stale(obj, [spath] + HEADERS):
            cmd = [hipcc] + HIPCC_FLAGS + ["-c", spath, "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    if force or procs or _stale(LIB, objs):
        cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
        subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    print(build_lib(force=True, verbose=True))
