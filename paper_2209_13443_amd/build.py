"""Builds libee.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libee.so")
SOURCES = ["kernels_conv.hip", "kernels_igemm.hip", "kernels_group.hip", "kernels_skinny.hip", "kernels_pair.hip", "kernels_seam.hip", "kernels_slab.hip", "kernels_rows.hip", "kernels_taps.hip", "kernels_thin.hip", "kernels_stream.hip", "kernels_ir.hip", "kernels_bneck.hip", "kernels_bneck16.hip", "kernels_stem.hip", "kernels_segment.hip", "kernels_misc.hip", "net.cpp", "ee_api.cpp", "serve.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",     # no packed-FP32 code generation
         "-Wall", "-Wno-unused-value", "-Wno-unused-function", "-Wno-unused-command-line-argument"]


def build(verbose=False):
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src + ".o")
        objs.append(obj)
        cmd = ["hipcc", *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd))
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
