"""Build libbwg.so in-tree for gfx950.

HIP sources are compiled by hipcc for gfx950, host-only C++ by g++ against
the HIP runtime headers (the binary128 Poisson tables need libquadmath).
The device headers that kernels compiled at run time include are embedded
as string constants in a generated source (_build/jit_headers.cpp).
Objects go to _build/ next to this file; the shared library lands in the
package directory, where the binding loads it.
"""

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INC = os.path.join(ROOT, "include")
OUT = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbwg.so")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

HIP_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17",
    # no packed-fp32 instructions anywhere in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + CSRC, "-I" + INC,
]
CXX_FLAGS = ["-O2", "-fPIC", "-std=gnu++17", "-D__HIP_PLATFORM_AMD__",
             "-I" + os.path.join(ROCM, "include"), "-I" + CSRC, "-I" + INC]


def _hipcc():
    p = shutil.which("hipcc") or os.path.join(ROCM, "bin", "hipcc")
    return p


def _compile(src):
    obj = os.path.join(OUT, os.path.basename(src) + ".o")
    if src.endswith(".hip"):
        cmd = [_hipcc(), "-c", src, "-o", obj] + HIP_FLAGS
    else:
        cmd = ["g++", "-c", src, "-o", obj] + CXX_FLAGS
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))
    return obj


# Headers of the device code that the run-time compiled kernels include.
JIT_HEADERS = ("bitops.h", "bwg_internal.h", "wm_device.h", "wm_event_body.inc", "event_draw.h",
               "lanes_device.h", "gen_device.h")


# The run-time compiler has the device builtins but no runtime header: the
# kernels see this stand-in, which only names the host types the headers'
# declarations mention.
JIT_RUNTIME_STUB = """#pragma once
#include <stdint.h>
typedef struct ihipStream_t *hipStream_t;
typedef int hipError_t;
"""


def _jit_headers_source():
    """Write _build/jit_headers.cpp: each header's text as a raw string."""
    delim = "BWG_JIT_HEADER"
    names = ("hip/hip_runtime.h",) + JIT_HEADERS
    parts = ["// generated by build.py from the device headers; do not edit",
             "namespace bwg {",
             "extern const int kJitHeaderCount = %d;" % len(names),
             "extern const char *const kJitHeaderNames[] = {%s};"
             % ", ".join('"%s"' % h for h in names),
             "extern const char *const kJitHeaders[] = {"]
    for h in names:
        if h == "hip/hip_runtime.h":
            text = JIT_RUNTIME_STUB
        else:
            with open(os.path.join(CSRC, h)) as f:
                text = f.read()
        if ")" + delim + '"' in text:
            raise RuntimeError("header %s contains the raw-string delimiter" % h)
        parts.append('R"%s(%s)%s",' % (delim, text, delim))
    parts += ["};", "}  // namespace bwg", ""]
    path = os.path.join(OUT, "jit_headers.cpp")
    with open(path, "w") as f:
        f.write("\n".join(parts))
    return path


def build(jobs=None, verbose=False):
    os.makedirs(OUT, exist_ok=True)
    srcs = sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC)
                  if f.endswith((".hip", ".cpp")))
    srcs.append(_jit_headers_source())
    jobs = jobs or min(8, os.cpu_count() or 1)
    with cf.ThreadPoolExecutor(jobs) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs + [
        "-lquadmath", "-L" + os.path.join(ROCM, "lib"), "-lhiprtc", "-lrocprofiler-sdk-roctx",
        "-Wl,-rpath," + os.path.join(ROCM, "lib")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))
    os.replace(tmp, LIB)
    _build_calib()
    if verbose:
        print("built", LIB)
    return LIB


CALIB_LIB = os.path.join(HERE, "libbwg_calib.so")
SELFTEST_LIB = os.path.join(HERE, "libbwg_selftest.so")
CPUGAIN_LIB = os.path.join(HERE, "libbwg_cpugain.so")


def _build_calib():
    """Small libraries of their own: the roofline reference kernels
    (calib/), the device self-test of the bit-sliced primitives (selftest/,
    used by the tests only) and the host-CPU engines of the paper's gain
    experiment (cpu_gain/, used by the benchmark only)."""
    for src, lib in ((os.path.join(HERE, "calib", "valu_ref.hip"), CALIB_LIB),
                     (os.path.join(HERE, "selftest", "prim_kernels.hip"), SELFTEST_LIB)):
        tmp = lib + ".tmp"
        cmd = [_hipcc(), "-shared", "-o", tmp, src] + HIP_FLAGS
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("compile failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))
        os.replace(tmp, lib)
    # the host-CPU engines of the paper's gain experiment (benchmark only)
    tmp = CPUGAIN_LIB + ".tmp"
    cmd = ["gcc", "-O3", "-shared", "-fPIC", "-std=c11", "-o", tmp,
           os.path.join(HERE, "cpu_gain", "gain_cpu.c")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))
    os.replace(tmp, CPUGAIN_LIB)


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
