"""Build libukst.so (HIP, gfx950) in-tree with hipcc.  Run: python -m paper_2502_20493_amd.build"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libukst.so")
MARSHAL_LIB = os.path.join(HERE, "_ukst_marshal.so")  # native marshalling of the Python binding
MARSHAL_SRC = os.path.join(CSRC, "binding", "ukst_marshal.cpp")
MARSHAL_STAMP = os.path.join(HERE, "_build", "marshal_built_for.txt")
BENCH_LIB = os.path.join(HERE, "libukst_bench.so")  # measurement helpers, not part of the product

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 VALU forms are kept off on purpose (scalar fp32 code only)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]
OBJDIR = os.path.join(HERE, "_build")


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def bench_sources():
    return sorted(glob.glob(os.path.join(CSRC, "bench", "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass warns that it does not know the packed-fp32 feature: harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(os.path.basename(cmd[0]) + " failed: " + " ".join(cmd) + "\n" + out)
    if verbose and out.strip():
        print(out)


def _marshal_command():
    """g++ line of the Python extension module that marshals tensors (CPython and torch headers, host code only)."""
    import sysconfig
    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DUKST_BUILT_FOR="{torch.__version__}"',
            "-I" + os.path.join(root, "include"), "-I" + os.path.join(rocm, "include"),
            "-I" + sysconfig.get_paths()["include"], MARSHAL_SRC, "-o", MARSHAL_LIB,
            "-L" + os.path.join(root, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]


def _marshal_versions():
    """What the extension module fits: this Python and this torch."""
    import torch
    return f"{sys.implementation.cache_tag} {torch.__version__}"


def build_library(verbose: bool = False, jobs: int | None = None) -> str:
    """Compile every csrc/*.hip to an object (in parallel) and link libukst.so; csrc/bench/*.hip
    become libukst_bench.so (the benchmark's measured ceilings), csrc/binding/ukst_marshal.cpp the binding's extension module."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJDIR, exist_ok=True)
    srcs, bsrcs = sources(), bench_sources()
    objs = [os.path.join(OBJDIR, os.path.basename(s)[:-4] + ".o") for s in srcs]
    bobjs = [os.path.join(OBJDIR, "bench_" + os.path.basename(s)[:-4] + ".o") for s in bsrcs]
    jobs = jobs or max(1, min(len(srcs), int(os.environ.get("MAX_JOBS", os.cpu_count() or 1)), 16))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        futs = [pool.submit(_run, [hipcc] + HIPCC_FLAGS + ["-c", s, "-o", o], verbose)
                for s, o in zip(srcs + bsrcs, objs + bobjs)]
        futs.append(pool.submit(_run, _marshal_command(), verbose))
        for f in futs:
            f.result()
    with open(MARSHAL_STAMP, "w") as f:
        f.write(_marshal_versions())
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + objs + ["-o", LIB], verbose)
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + bobjs + ["-o", BENCH_LIB], verbose)
    return LIB


def is_stale() -> bool:
    libs = (LIB, BENCH_LIB, MARSHAL_LIB)
    if not all(os.path.exists(p) for p in libs + (MARSHAL_STAMP,)):
        return True
    with open(MARSHAL_STAMP) as f:
        if f.read() != _marshal_versions():
            return True
    t = min(os.path.getmtime(p) for p in libs)
    deps = sources() + bench_sources() + [MARSHAL_SRC] + glob.glob(os.path.join(CSRC, "*.h")) + \
        glob.glob(os.path.join(HERE, "..", "include", "*.h"))
    return any(os.path.getmtime(d) > t for d in deps)


if __name__ == "__main__":
    print(build_library(verbose=True))
    sys.exit(0)
