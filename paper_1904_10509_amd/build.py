"""Compile the HIP library libsparse_attn.so for gfx950, in-tree.

Every source under csrc/ is compiled with hipcc into _build/ and linked into
paper_1904_10509_amd/libsparse_attn.so next to this file.  The benchmark's
measurement probe (probe/*.hip, the matrix-core peak and clock) becomes
libsa_probe.so beside it.
"""
import concurrent.futures as cf
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(os.path.dirname(HERE), "_build")
LIB = os.path.join(HERE, "libsparse_attn.so")
PROBE_DIR = os.path.join(HERE, "probe")
PROBE_LIB = os.path.join(HERE, "libsa_probe.so")
ARCH = "gfx950"
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Packed fp32 VALU instructions are kept out of generated code on purpose.
# MFMA results stay in ordinary VGPRs (the softmax works on them directly),
# and maxima skip NaN quieting: the kernels never produce NaNs from finite
# inputs, and what attends an infinity or a NaN is unspecified (tests for one
# look at the bits: csrc/sa_finite.h).
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-mfma-vgpr-form=1", "-fno-honor-nans",
         "-I", os.path.join(os.path.dirname(HERE), "include")]


# Per-source additions.  The forward kernels keep their O accumulators in
# the same registers across the two ring stages and the masked and unmasked
# step bodies only when copies on split edges and across blocks are
# coalesced (about ten 64-bit moves fewer per step; the forward at n = 12,288
# dense 0.406 -> 0.390 ms).  The backward kernels measured 1-3% slower with
# the same options, so they keep the defaults.
FILE_FLAGS = {"sa_fwd.hip": ["-mllvm", "-join-globalcopies=true", "-mllvm", "-join-splitedges=true"]}


def sources(folder=CSRC):
    return sorted(os.path.join(folder, f) for f in os.listdir(folder) if f.endswith(".hip"))


def _compile(src):
    obj = os.path.join(BUILD, os.path.basename(os.path.dirname(src)) + "_" + os.path.basename(src) + ".o")
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = [ln for ln in (r.stdout + r.stderr).splitlines()
            if "packed-fp32-ops' is not a recognized feature" not in ln]
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n" + "\n".join(msgs))
    return obj, "\n".join(msgs)


def _link(objs, lib):
    tmp = lib + ".tmp"
    subprocess.run([HIPCC, "-shared", f"--offload-arch={ARCH}", "-o", tmp, *objs], check=True)
    os.replace(tmp, lib)


def build(verbose: bool = False) -> str:
    """Compile every csrc/*.hip and probe/*.hip and link the two shared
    libraries; returns the attention library's path."""
    os.makedirs(BUILD, exist_ok=True)
    lib_srcs, probe_srcs = sources(CSRC), sources(PROBE_DIR)
    with cf.ThreadPoolExecutor(max_workers=min(9, os.cpu_count() or 1)) as ex:
        results = list(ex.map(_compile, lib_srcs + probe_srcs))
    for obj, msgs in results:
        if verbose and msgs.strip():
            print(msgs)
    objs = [o for o, _ in results]
    _link(objs[: len(lib_srcs)], LIB)
    _link(objs[len(lib_srcs):], PROBE_LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
