"""Builds liblasnet.so (HIP, gfx950 only) in-tree with hipcc.  `python -m paper_2210_06223_amd.build`."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "liblasnet.so")
# The check build: the same sources with every hand-counted barrier of the matrix-core kernels waiting
# for all outstanding memory operations.  Only the tests load it (to compare the two bit for bit).
LIB_CHECK = os.path.join(PKG, "liblasnet_check.so")
CHECK_FLAGS = ("-DLASNET_DRAIN_AT_BARRIERS",)
# The binding's native argument marshalling: host code against torch's headers, no HIP in it.
MARSHAL = os.path.join(PKG, "_marshal.so")
SOURCES = ["tiled_stages.hip", "mfma_stage3.hip", "mfma_stage2.hip", "mfma_stage1.hip", "mfma_stage4.hip",   # slowest first
           "rows_generic.hip", "slab_stages.hip",
           "api.hip", "masker.hip", "bottleneck_generic.hip", "bottleneck_mfma.hip", "microbench.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU ops
    "-Wno-unused-command-line-argument", "-Wno-unknown-attributes",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


# The k-loops of the matrix-core kernels must be unrolled in full (their register rings are indexed
# by the loop counter, and the counts of their barriers are worked out from it: a loop that is not unrolled
# keeps its ring in scratch memory and picks each count at run time).  The long reductions of the tiled
# kernels and of the fused kernel at 2048 channels exceed the compiler's default size limit for `#pragma unroll`.
PER_FILE_FLAGS = {f: ["-mllvm", "-pragma-unroll-threshold=1048576"] for f in ("tiled_stages.hip", "mfma_stage4.hip")}


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: liblasnet cannot be built")
    return exe


def _compile(cc, src, obj, extra_flags, verbose):
    cmd = [cc, *FLAGS, *PER_FILE_FLAGS.get(src, []), *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return obj


def _link(cc, objs, out, verbose):
    tmp = out + ".tmp"
    r = subprocess.run([cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, out)
    if verbose:
        print("built", out)
    return out


def build_variants(variants, verbose: bool = True) -> None:
    """variants: (output path, build directory, extra flags) each; all files of all variants are
    compiled through one pool of workers, then each variant is linked."""
    cc = hipcc()
    jobs = []
    for out, bdir, extra in variants:
        os.makedirs(bdir, exist_ok=True)
        for src in SOURCES:
            jobs.append((src, os.path.join(bdir, os.path.splitext(src)[0] + ".o"), tuple(extra)))
    jobs.sort(key=lambda j: SOURCES.index(j[0]))          # slowest files first, over all variants
    with ThreadPoolExecutor(max_workers=min(8, len(jobs), os.cpu_count() or 1)) as ex:
        list(ex.map(lambda j: _compile(cc, j[0], j[1], j[2], verbose), jobs))
    for out, bdir, _ in variants:
        _link(cc, [os.path.join(bdir, os.path.splitext(src)[0] + ".o") for src in SOURCES], out, verbose)


def build_library(verbose: bool = True, extra_flags=(), out: str = LIB, build_dir: str = "") -> str:
    build_variants([(out, build_dir or os.path.join(PKG, "_build"), extra_flags)], verbose)
    return out


def build_marshal(verbose: bool = True) -> str:
    import sysconfig
    import torch
    inc, lib = (os.path.join(os.path.dirname(torch.__file__), d) for d in ("include", "lib"))
    tmp = MARSHAL + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           "-I" + inc, "-I" + os.path.join(inc, "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
           "-I" + os.path.join(ROOT, "include"), os.path.join(CSRC, "marshal.cpp"), "-o", tmp,
           "-L" + lib, "-Wl,-rpath," + lib, "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed on marshal.cpp:\n" + r.stderr)
    os.replace(tmp, MARSHAL)
    if verbose:
        print("built", MARSHAL)
    return MARSHAL


def build_all(verbose: bool = True) -> None:
    with ThreadPoolExecutor(max_workers=1) as ex:
        marshal = ex.submit(build_marshal, verbose)
        build_variants([(LIB, os.path.join(PKG, "_build"), ()),
                        (LIB_CHECK, os.path.join(PKG, "_build", "check"), CHECK_FLAGS)], verbose)
        marshal.result()


if __name__ == "__main__":
    build_all()
