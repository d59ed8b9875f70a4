"""Build of the HIP library (libforkstep.so) for gfx950.

``python -m paper_2609_39859_amd.build`` compiles the library's HIP sources
under csrc/ with hipcc into libforkstep.so next to this file, and the
benchmark's peak probes (csrc/peak_probe.hip) into libforkprobe.so, and with
g++ the Python binding's native calls into _fastcall.so.  The hipcc compile
disables packed-fp32 instruction selection (the -packed-fp32-ops target
feature); hipcc's host pass warns that it does not know the feature, which is
harmless.
"""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libforkstep.so")
SOURCES = ["gemm_stats.hip", "gemm_narrow.hip", "gemm_f32.hip",
           "merge_select.hip", "grpo.hip", "fork_abi.hip"]
PROBE_LIB = os.path.join(HERE, "libforkprobe.so")
PROBE_SOURCES = ["peak_probe.hip"]
ARCH = "gfx950"


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    return "hipcc"


def compile_flags():
    return ["-std=c++17", "-O3", "-fPIC", "--offload-arch=%s" % ARCH,
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-result", "-I", INCLUDE, "-I", CSRC]


def build(verbose: bool = False) -> str:
    """Compile and link libforkstep.so and libforkprobe.so, then the plain-C
    example that drives one step through the C ABI; returns the path of
    libforkstep.so.  The binding works without _fastcall.so: if that cannot be
    compiled a warning says so and none is left in place."""
    fast = _start_fastcall(verbose)
    try:
        _build_lib(PROBE_LIB, PROBE_SOURCES, verbose)
        lib = _build_lib(LIB, SOURCES, verbose)
    except BaseException:
        _finish_fastcall(fast, install=False)
        raise
    _finish_fastcall(fast, install=True)
    build_c_example(verbose)
    return lib


FASTCALL = os.path.join(HERE, "_fastcall.so")


def _start_fastcall(verbose: bool = False):
    """Start the host compile of _fastcall.so (csrc/fastcall.cpp: the Python
    binding's plain calls, against torch's headers); _finish_fastcall() ends
    it.  None if there is no compiler or no torch."""
    import sysconfig
    try:
        import torch
        from torch.utils.cpp_extension import include_paths
        libdir = os.path.join(os.path.dirname(torch.__file__), "lib")
        tmp = FASTCALL + ".tmp%d" % os.getpid()
        cmd = ["g++", "-std=c++17", "-O2", "-fPIC", "-shared", "-Wall", "-I", INCLUDE,
               "-I", sysconfig.get_paths()["include"],
               "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI)]
        for inc in include_paths():
            cmd += ["-isystem", inc]
        cmd += [os.path.join(CSRC, "fastcall.cpp"), "-L", libdir, "-ltorch_python", "-ltorch_cpu",
                "-lc10", "-o", tmp]
        if verbose:
            print(" ".join(cmd), flush=True)
        return subprocess.Popen(cmd), tmp
    except (ImportError, OSError) as e:
        print("_fastcall.so: %s" % e, file=sys.stderr)
        return None


def _finish_fastcall(job, install: bool) -> None:
    """Wait for the compile; put its result in place (install) or drop it.
    Without a result the one in place, made for another library, goes too."""
    ok = job is not None and job[0].wait() == 0
    if ok and install:
        os.replace(job[1], FASTCALL)
        return
    if job is not None and os.path.exists(job[1]):
        os.remove(job[1])
    if install:
        if os.path.exists(FASTCALL):
            os.remove(FASTCALL)
        print("warning: fastcall.cpp was not compiled; calls go through ctypes", file=sys.stderr)


C_EXAMPLE_SRC = os.path.join(ROOT, "tests", "native", "abi_c_step.c")
C_EXAMPLE = os.path.join(HERE, "_build", "abi_c_step")


def build_c_example(verbose: bool = False) -> str:
    """gcc -std=c99 build of tests/native/abi_c_step.c against the public
    header, libforkstep.so and the HIP runtime's C API."""
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    os.makedirs(os.path.dirname(C_EXAMPLE), exist_ok=True)
    cmd = ["gcc", "-std=c99", "-O1", "-Wall", "-Wextra", "-Werror", "-D__HIP_PLATFORM_AMD__",
           "-I", os.path.join(rocm, "include"), "-I", INCLUDE, C_EXAMPLE_SRC,
           "-L", HERE, "-lforkstep", "-L", os.path.join(rocm, "lib"), "-lamdhip64", "-lm",
           "-Wl,-rpath,$ORIGIN/..", "-o", C_EXAMPLE]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return C_EXAMPLE


def _build_lib(lib_path: str, sources, verbose: bool) -> str:
    objs = []
    builddir = os.path.join(HERE, "_build")
    os.makedirs(builddir, exist_ok=True)
    procs = []
    for src in sources:
        obj = os.path.join(builddir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc()] + compile_flags() + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE,
                                            stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    failed = []
    for src, p in procs:
        out, _ = p.communicate()
        # the host pass's note about the packed-fp32 feature is expected noise
        lines = [ln for ln in out.splitlines() if "packed-fp32-ops" not in ln]
        if lines and (verbose or p.returncode):
            print("\n".join(lines), file=sys.stderr)
        if p.returncode:
            failed.append(src)
    if failed:
        raise RuntimeError("hipcc failed for %s" % ", ".join(failed))
    tmp = lib_path + ".tmp%d" % os.getpid()
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=%s" % ARCH, "-o", tmp] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, lib_path)
    return lib_path


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
