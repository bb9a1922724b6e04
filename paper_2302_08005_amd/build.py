"""Compiles the HIP sources into libslapo_mi355x.so next to this file (gfx950 only)."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libslapo_mi355x.so")
SOURCES = ("api.hip", "gemm.hip", "grads.hip", "products.hip", "attention.hip", "rowwise.hip")
# per-file extra flags: the attention kernels alternate MFMA and vector work on the same tiles, so their MFMA
# results are kept in ordinary VGPRs (the default puts them in accumulation registers and copies them back
# and forth for every softmax)
EXTRA = {"attention.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}
# kernels start on pages of 4 KB: a step launches a different one each time, whose code is fetched anew, and every page that it touches
# costs. Three decoder layers of 72 tokens, hidden 1088, backward, with kernels on 256 / 1024 / 2048 / 4096 bytes: 185.9 / 185.1 / 184.3 /
# 182.5 us; an encoder layer of 2 x 824 tokens, hidden 384, checkpointed, 192.8 / 190.9 / 191.1 / 191.0. (5 MB of padding.)
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-falign-functions=4096", "-Xclang", "-target-feature", "-Xclang",
         "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


def build(verbose: bool = True) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc] + FLAGS + EXTRA.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out, file=sys.stderr)
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs)
    return LIB


if __name__ == "__main__":
    print(build())
