"""Build libntp.so (HIP kernels + C boundary) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libntp.so")
PROBE_SRC = os.path.join(CSRC, "line_rate_probe.hip")
PROBE = os.path.join(PKG, "line_rate_probe")        # prints the chip's 128-byte line rates (L2 / Infinity Cache / HBM)

NATIVE_SRC = os.path.join(CSRC, "py_native.cpp")
NATIVE = os.path.join(PKG, "_native" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))       # Python entry to the enqueue calls

SOURCES = ["graph_build.cpp", "graph_device.hip", "plan.cpp", "ntp_api.hip", "agg_kernels.hip", "scatter_kernels.hip", "chunk_kernels.hip", "attention_kernels.hip", "attention_scores_kernels.hip", "loss_kernels.hip", "nn_kernels.hip", "nn_strip_kernels.hip", "nn_resident_kernels.hip", "nn_dw_kernels.hip"]
HEADERS = [os.path.join(CSRC, "ntp_internal.h"), os.path.join(CSRC, "lane_util.h"), os.path.join(CSRC, "nn_util.h"), os.path.join(CSRC, "chunk_schedule.h"), os.path.join(CSRC, "row_copies.h"), os.path.join(CSRC, "entry_export.h"), os.path.join(ROOT, "include", "ntp.h")]

COMMON = ["-O3", "-std=c++17", "-fPIC", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
          "-ffp-contract=off", "-Wall", "-Wno-unused-function"]
# packed fp32 instructions (v_pk_*_f32) are switched off for device code: the compiler must
# not form them from ordinary float arithmetic
DEVICE = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    raise RuntimeError("hipcc not found")


def _stale(out: str, deps) -> bool:
    if not os.path.exists(out):
        return True
    t = os.path.getmtime(out)
    return any(os.path.getmtime(d) > t for d in deps)


def native_command(out: str):
    """Compiler line of the Python entry module, or None where the interpreter's headers are missing (the binding then
    marshals with ctypes)."""
    include = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(include, "Python.h")):
        return None
    cxx = [shutil.which("g++")] if shutil.which("g++") else [_hipcc(), "-x", "c++"]
    return cxx + ["-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I" + os.path.join(ROOT, "include"), "-I" + include, NATIVE_SRC,
                  "-o", out, "-L" + PKG, "-lntp", "-Wl,-rpath,$ORIGIN"]


def build(force: bool = False, verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    hipcc = _hipcc()
    jobs = []
    for s in SOURCES:
        src = os.path.join(CSRC, s)
        obj = os.path.join(OBJ, s + ".o")
        if force or _stale(obj, [src] + HEADERS):
            cmd = [hipcc, "-c", "-x", "hip", src, "-o", obj] + COMMON + DEVICE
            jobs.append(cmd)

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        if r.returncode != 0:
            raise RuntimeError("compile failed:\n%s\n%s" % (" ".join(cmd), r.stdout))
        return r.stdout

    with ThreadPoolExecutor(max_workers=min(8, max(1, len(jobs)))) as ex:
        for out in ex.map(run, jobs):
            if verbose and out.strip():
                print(out)
    objs = [os.path.join(OBJ, s + ".o") for s in SOURCES]
    if force or jobs or _stale(LIB, objs):
        tmp = LIB + ".tmp%d" % os.getpid()
        run([hipcc, "-shared", "-fPIC", "-o", tmp] + objs + ["--offload-arch=gfx950", "-lpthread"])
        os.replace(tmp, LIB)
    if force or _stale(NATIVE, [NATIVE_SRC, os.path.join(ROOT, "include", "ntp.h"), os.path.abspath(__file__)]):
        tmp = NATIVE + ".tmp%d" % os.getpid()
        cmd = native_command(tmp)
        if cmd:
            run(cmd)
            os.replace(tmp, NATIVE)
        elif verbose:
            print("no Python.h: calls go through ctypes")
    # the stand-alone measurement aid (its own executable: it links nothing of the library)
    if force or _stale(PROBE, [PROBE_SRC]):
        tmp = PROBE + ".tmp%d" % os.getpid()
        run([hipcc, "-O3", "-std=c++17", "-ffp-contract=off", "-o", tmp, PROBE_SRC] + DEVICE)
        os.replace(tmp, PROBE)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv, verbose=True))
