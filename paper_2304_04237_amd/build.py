"""Build libslide_attn.so (HIP, gfx950 only) in-tree with hipcc.

Run `python -m paper_2304_04237_amd.build`.  The shared object lands next to
this file; it is git-ignored but travels with the tree to the GPU machine.
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libslide_attn.so")
SOURCES = ["slide_api.hip", "slide_generic.hip", "slide_mfma32.hip", "slide_mfma32_bwd.hip", "slide_split.hip", "slide_split_dw.hip", "slide_fwd16.hip", "slide_fwd16_ring.hip", "slide_bwd_dw.hip", "slide_bwd16.hip", "slide_bwd16_ring.hip", "slide_fwd16_k5.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def build(verbose=False):
    flags = FLAGS + os.environ.get("SLIDE_ATTN_EXTRA_HIPCC_FLAGS", "").split()   # e.g. -D switches of development builds
    objs = []
    build_dir = os.path.join(HERE, "_build")
    os.makedirs(build_dir, exist_ok=True)
    procs = []
    for src in SOURCES:
        obj = os.path.join(build_dir, src.replace(".hip", ".o"))
        cmd = ["hipcc"] + flags + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, pr in procs:
        out, _ = pr.communicate()
        # the host pass does not know the packed-fp32 feature name; that notice is harmless
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if pr.returncode != 0:
            raise RuntimeError("hipcc failed on %s:\n%s" % (src, out))
        if verbose and out.strip():
            print(out)
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
