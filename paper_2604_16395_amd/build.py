"""Build libs2l.so (HIP kernels for gfx950 + the C-ABI layer) and the Python package's native
argument marshalling (_binding.*.so, CPython API; only where Python's headers are) in place.

Usage: python -m paper_2604_16395_amd.build [-v] [--sanitize]

--sanitize also builds _build/san/libs2l.so: the same device objects, with the host C++
(argument validation, the host planner, the scheduler) compiled by g++ under AddressSanitizer
and UndefinedBehaviorSanitizer.  Load it with S2L_LIBRARY=<path> and the ASan runtime first in
LD_PRELOAD (tests/test_sanitize_cpu.py runs the host-side test files that way); it is for the
CPU tests, not for GPU runs.
"""
import concurrent.futures
import glob
import os
import shutil
import subprocess
import sys
import sysconfig
import warnings

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libs2l.so")
# named for the interpreter it is built for, so that another one does not take it
BINDING = os.path.join(PKG, "_binding" + sysconfig.get_config_var("EXT_SUFFIX"))
ARCH = "gfx950"


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


COMMON = ["-O3", "-fPIC", "-std=c++17", "-I", INCLUDE, "-I", CSRC, "-Wall", "-Wno-unused-result"]
# No packed fp32 ops in device code (v_pk_*_f32 are avoided on this hardware).
DEVICE = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-munsafe-fp-atomics"]
# The attention kernels' first arguments (14 dwords) arrive in registers instead of through a load
# that the item's address waits for: 0.15 to 0.3 us of a launch.  Setting the registers up costs 0.1
# us, more than the page kernels' shorter chains gain (append of one row 2.10 us without, 2.24 with).
PRELOAD = {"chunk_attn.hip", "decode_attn.hip"}
PRELOAD_FLAGS = ["-mllvm", "-amdgpu-kernarg-preload-count=14"]


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    p = subprocess.run(cmd, capture_output=True, text=True)
    out = "\n".join(l for l in (p.stdout + p.stderr).splitlines()
                    if "packed-fp32-ops" not in l and l.strip())
    if p.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{out}")
    if verbose and out:
        print(out)
    return cmd[-1]


def build(verbose=False):
    os.makedirs(BUILD, exist_ok=True)
    hipcc = _hipcc()
    jobs = []
    for src in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        obj = os.path.join(BUILD, os.path.basename(src) + ".o")
        extra = PRELOAD_FLAGS if os.path.basename(src) in PRELOAD else []
        jobs.append([hipcc, "-x", "hip", *COMMON, *DEVICE, *extra, "-c", src, "-o", obj])
    for src in sorted(glob.glob(os.path.join(CSRC, "*.cpp"))):
        obj = os.path.join(BUILD, os.path.basename(src) + ".o")
        jobs.append([hipcc, *COMMON, "-c", src, "-o", obj])
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(jobs))) as ex:
        objs = list(ex.map(lambda cmd: _run(cmd, verbose), jobs))
    tmp = LIB + ".tmp"
    _run([hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs], verbose)
    os.replace(tmp, LIB)
    build_binding(verbose)
    return LIB


def build_binding(verbose=False):
    """The _binding module for the running interpreter.  Without Python's headers there is none (one of an
    earlier build is removed, as it may follow another s2l.h): the package then marshals all its
    calls through ctypes, and the library itself does not need it."""
    headers = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(headers, "Python.h")):
        warnings.warn(f"no Python.h in {headers}: {os.path.basename(BINDING)} is not built, calls marshal through ctypes")
        if os.path.exists(BINDING):
            os.remove(BINDING)
        return None
    _run([_hipcc(), *COMMON, "-shared", "-I", headers, os.path.join(CSRC, "python", "binding.cpp"),
          "-o", BINDING + ".tmp"], verbose)
    os.replace(BINDING + ".tmp", BINDING)
    return BINDING


SAN = os.path.join(BUILD, "san")
SAN_LIB = os.path.join(SAN, "libs2l.so")
SAN_FLAGS = ["-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-fno-omit-frame-pointer"]


def build_sanitized(verbose=False):
    """Host sources under ASan + UBSan (g++), linked with the device objects of build(), and, where
    Python's headers are, the native marshalling likewise, beside the library."""
    build(verbose)
    os.makedirs(SAN, exist_ok=True)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(_hipcc())))
    gxx = os.environ.get("CXX") or shutil.which("g++")
    if not gxx:
        raise RuntimeError("g++ not found")
    objs = []
    for src in sorted(glob.glob(os.path.join(CSRC, "*.cpp"))):
        obj = os.path.join(SAN, os.path.basename(src) + ".o")
        cmd = [gxx, "-std=c++17", "-O1", "-g", "-fPIC", *SAN_FLAGS, "-D__HIP_PLATFORM_AMD__",
               "-I", os.path.join(rocm, "include"), "-I", INCLUDE, "-I", CSRC, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        objs.append(obj)
    dev = sorted(glob.glob(os.path.join(BUILD, "*.hip.o")))
    lib_dir = os.path.join(rocm, "lib")
    cmd = [gxx, "-shared", *SAN_FLAGS, "-o", SAN_LIB, *dev, *objs, "-L", lib_dir, "-lamdhip64",
           f"-Wl,-rpath,{lib_dir}"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    headers = sysconfig.get_paths()["include"]
    if os.path.exists(os.path.join(headers, "Python.h")):
        cmd = [gxx, "-std=c++17", "-O1", "-g", "-fPIC", "-shared", *SAN_FLAGS, "-I", headers, "-I", INCLUDE,
               os.path.join(CSRC, "python", "binding.cpp"), "-o", os.path.join(SAN, os.path.basename(BINDING))]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
    return SAN_LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
    if "--sanitize" in sys.argv:
        print(build_sanitized(verbose="-v" in sys.argv))
