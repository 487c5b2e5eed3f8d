"""Builds liboxy.so (HIP kernels for gfx950 + host pool) in-tree with hipcc."""
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liboxy.so")
SOURCES = ["oxy_kernels.hip", "oxy_pool.cpp", "oxy_sched.cpp"]
# packed fp32 VALU forms are switched off for device code on purpose; the first eight arguments of a
# kernel (at most 14 words, none from a struct on) are preloaded into scalar registers
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                "-mllvm", "-amdgpu-kernarg-preload-count=8"]


PROBE_SRC = os.path.join(HERE, "benchaid", "probe_kernels.hip")
PROBE_LIB = os.path.join(HERE, "benchaid", "libprobe.so")


MARSHAL_SRC = os.path.join(CSRC, "oxy_python.cpp")
MARSHAL_LIB = os.path.join(HERE, "libmarshal.so")


def _compile(compiler, flags, sources, target, verbose):
    cmd = [compiler, "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unused-result"]
    cmd += list(flags) + list(sources) + ["-o", target]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines()
                    if "packed-fp32-ops' is not a recognized feature" not in l)
    if res.returncode != 0:
        raise RuntimeError("%s failed:\n%s" % (compiler, out))
    if verbose and out.strip():
        print(out)
    return target


def build_library(verbose=False):
    """liboxy.so (the method), benchaid/libprobe.so (the benchmark's measurement aids) and, where
    Python's headers and a host compiler are there, libmarshal.so (list conversion of the Python
    binding, which converts by Python's own means without it)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _compile(hipcc, DEVICE_FLAGS, [os.path.join(CSRC, s) for s in SOURCES], LIB, verbose)
    _compile(hipcc, DEVICE_FLAGS, [PROBE_SRC], PROBE_LIB, verbose)
    headers, cxx = sysconfig.get_paths()["include"], os.environ.get("CXX", "g++")
    if os.path.exists(os.path.join(headers, "Python.h")) and shutil.which(cxx):
        _compile(cxx, ["-I" + headers], [MARSHAL_SRC], MARSHAL_LIB, verbose)   # no HIP in it
    else:
        if os.path.exists(MARSHAL_LIB):
            os.remove(MARSHAL_LIB)   # of an earlier build, maybe for another Python
        if verbose:
            print("libmarshal.so not built: no Python.h in %s or no %s" % (headers, cxx))
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
    sys.exit(0)
