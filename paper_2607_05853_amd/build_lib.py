"""Build libbse.so (gfx950) from the HIP sources in csrc/.

Every source is compiled for gfx950 only, with packed FP32 instructions
disabled, and linked into one shared library next to this file.
"""
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libbse.so")
SOURCES = ["api.hip", "gemm.hip", "interp.hip", "apply.hip", "direct_b3.hip", "lanczos.hip", "lobpcg.hip",
           "util.hip", "full.hip", "noalloc.hip", "fourier.hip",
           "lattice.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-result", "-I" + os.path.join(HERE, "..", "include")]


def build(verbose=False, jobs=None):
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs, objs = [], []
    for s in SOURCES:
        src = os.path.join(CSRC, s)
        obj = os.path.join(objdir, s.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((s, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
    failed = []
    for s, p in procs:
        out, _ = p.communicate()
        txt = out.decode(errors="replace")
        if p.returncode != 0:
            failed.append((s, txt))
        elif verbose and txt.strip():
            print(txt)
    if failed:
        for s, txt in failed:
            sys.stderr.write("=== %s ===\n%s\n" % (s, txt))
        raise RuntimeError("HIP compilation failed: " + ", ".join(s for s, _ in failed))
    tmp = OUT + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs
    subprocess.check_call(cmd)
    shutil.move(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
