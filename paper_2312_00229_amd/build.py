"""Build the HIP library in-tree: hipcc for gfx950 -> paper_2312_00229_amd/libweno_zoom.so,
and the binding's call path, gcc -> _native.so.

Flags: -O3, FP contraction off (every fused multiply-add in the kernels is
written explicitly, so the operation sequence -- and hence every bit of the
result -- is the same in all kernels that share the device code), packed FP32
disabled, C++17."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libweno_zoom.so")
NATIVE = os.path.join(PKG, "_native.so")   # the binding's call path (CPython extension)
# (source, macros, object name): the doubling's kernels compile once per I/O
# mode (kIo* of weno_fwd.h), so that the compilations run side by side
OBJECTS = [("weno_zoom.hip", ["-DWENO_IO=%d" % io], "weno_zoom%d" % io) for io in range(8)] + [
    ("weno_api.hip", [], "weno_api"), ("weno_bwd.hip", [], "weno_bwd"), ("weno_resample.hip", [], "weno_resample")]
ARCH = os.environ.get("WENO_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build the library)")


DEVICE_FLAGS = ["--offload-arch=" + ARCH, "-std=c++17", "-fPIC", "-ffp-contract=off",
                "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-result",
                "-I" + INCLUDE, "-I" + CSRC]


def _compile(flags, out_dir, verbose):
    """The objects of OBJECTS in out_dir, a few compilations at a time."""
    jobs = int(os.environ.get("MAX_JOBS") or min(8, os.cpu_count() or 1))

    def one(entry):
        src, macros, name = entry
        obj = os.path.join(out_dir, name + ".o")
        cmd = [hipcc(), *flags, *DEVICE_FLAGS, *macros, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            sys.stderr.write(res.stdout + res.stderr)
            raise RuntimeError("hipcc failed compiling %s" % src)
        return obj

    with ThreadPoolExecutor(max(1, jobs)) as pool:
        return list(pool.map(one, OBJECTS))


def build_native(verbose: bool = False) -> str:
    tmp = NATIVE + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CC") or "gcc", "-O2", "-shared", "-fPIC", "-Wall", "-I" + sysconfig.get_paths()["include"],
           "-I" + INCLUDE, os.path.join(CSRC, "weno_native.c"), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("building %s failed" % NATIVE)
    os.replace(tmp, NATIVE)
    return NATIVE


def build(verbose: bool = False) -> str:
    build_native(verbose)
    tmp = LIB + ".tmp%d" % os.getpid()
    with tempfile.TemporaryDirectory() as objs_dir:
        objs = _compile(["-O3"], objs_dir, verbose)
        cmd = [hipcc(), "--offload-arch=" + ARCH, "-shared", "-fPIC", *objs, "-o", tmp]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError("hipcc failed building %s" % LIB)
    os.replace(tmp, LIB)
    return LIB


def build_asan(out_dir: str, verbose: bool = False) -> str:
    """The same library with AddressSanitizer on its HOST code only (device
    code is built as usual), for the ABI checks on the CPU, linked into
    out_dir/libweno_zoom_asan.so.  Load it through WENO_ZOOM_LIB with the
    sanitizer runtime preloaded (asan_runtime())."""
    os.makedirs(out_dir, exist_ok=True)
    objs = _compile(["-O1", "-g", "-fno-omit-frame-pointer", "-Xarch_host", "-fsanitize=address"], out_dir, verbose)
    lib = os.path.join(out_dir, "libweno_zoom_asan.so")
    cmd = [hipcc(), "--offload-arch=" + ARCH, "-shared", "-fPIC", "-Xarch_host", "-fsanitize=address", *objs,
           "-o", lib]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True, capture_output=True)
    return lib


def asan_runtime() -> str:
    """Path of the AddressSanitizer runtime of ROCm's clang."""
    clang = os.path.join(os.path.dirname(os.path.realpath(hipcc())), "..", "lib", "llvm", "bin", "clang")
    if not os.path.exists(clang):
        clang = "/opt/rocm/llvm/bin/clang"
    res = subprocess.run([clang, "--print-file-name=libclang_rt.asan-x86_64.so"], capture_output=True, text=True,
                         check=True)
    return res.stdout.strip()


if __name__ == "__main__":
    print(build(verbose=True))
