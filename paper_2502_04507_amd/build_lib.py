"""Build libsta.so (the C-ABI HIP library) and libsta_mfma_probe.so (a matrix-instruction-only kernel that the
benchmark alone loads) for gfx950 with hipcc, and sta_fastcall.so (the CPython extension that calls the library's hot entry
points) with the host compiler, in-tree."""
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libsta.so")
BUILD_DIR = os.path.join(HERE, "_build")
SOURCES = ["sta_api.hip", "sta_permute.hip", "sta_attention.hip", "sta_reduce.hip", "sta_backward.hip"]
PROBE_SOURCE = "bench_mfma_probe.hip"
PROBE_OUT = os.path.join(HERE, "libsta_mfma_probe.so")

FASTCALL_SOURCE = "sta_fastcall.cpp"
FASTCALL_OUT = os.path.join(HERE, "sta_fastcall.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    # no NaN is ever produced inside the kernels (the only infinities are the initial running maxima, which meet
    # finite values only); saying so lets max chains compile to v_max3_f32 without per-operand canonicalisation
    "-fno-honor-nans",
    # matrix instructions accumulate in vector registers everywhere.  Left to itself the compiler moves the accumulators of
    # kernels whose LDS allows one wave per SIMD into accumulation registers and copies them to scale or test them (40 heads of
    # 64x96 in 32-token tiles, head dimension 128: forward 118 -> 97 us, gradients 232 -> 221)
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    noise = "is not a recognized feature for this target"
    warn = "\n".join(l for l in r.stderr.splitlines() if l.strip() and noise not in l)
    if warn:
        sys.stderr.write(warn + "\n")
    return obj


def _build_fastcall() -> str:
    """Builds the extension; returns what went wrong, or an empty string.  It needs a host compiler and the headers of Python and
    torch, which the library does not, and the package works without it."""
    import torch
    root = os.path.dirname(torch.__file__)
    include, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-isystem", include, "-isystem",
           os.path.join(include, "torch", "csrc", "api", "include"), "-I", sysconfig.get_paths()["include"],
           os.path.join(CSRC, FASTCALL_SOURCE), "-o", FASTCALL_OUT, "-L", lib, "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-Wl,-rpath," + lib]
    if os.path.exists(FASTCALL_OUT):
        os.remove(FASTCALL_OUT)                     # never one that the present sources did not make
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
    except OSError as e:
        return "%s: %s" % (cmd[0], e)
    return "" if r.returncode == 0 else r.stdout + r.stderr


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=len(SOURCES) + 2) as ex:
        fastcall = ex.submit(_build_fastcall)
        objs = list(ex.map(_compile, SOURCES + [PROBE_SOURCE]))
        missing = fastcall.result()
    for out, members in ((OUT, objs[:-1]), (PROBE_OUT, objs[-1:])):
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", out] + members
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
        if verbose:
            print(out)
    if missing:
        sys.stderr.write("%s was not built; libsta.so is there and is called through ctypes:\n%s\n" % (FASTCALL_OUT, missing))
    elif verbose:
        print(FASTCALL_OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
