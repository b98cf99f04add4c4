"""Build libifq.so (HIP for gfx950 + host C++) and the extension module _ifqcall
(the CPython entry to its launching functions, for the interpreter that runs
this) into this package directory. Needs hipcc, a C compiler and Python.h.

Usage: python paper_1911_08076_amd/build.py (runs without importing the
package, which needs the library to exist)
"""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libifq.so")
# the interpreter's own suffix: another Python does not take the module for its own
CALL = os.path.join(HERE, "_ifqcall" + sysconfig.get_config_var("EXT_SUFFIX"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

SOURCES = ["ifq_api.cpp", "ifq_conv.hip", "ifq_conv_mfma.hip", "ifq_conv_halo.hip", "ifq_conv_w2.hip", "ifq_conv_wp.hip", "ifq_conv_win.hip",
           "ifq_noalloc.hip",
           "ifq_conv_small.hip", "ifq_pool.hip", "ifq_thresholds.hip"]


def build(verbose=False):
    """Compile every source to an object in parallel, then link libifq.so."""
    from concurrent.futures import ThreadPoolExecutor
    flags = [HIPCC, "--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC",
             "-fvisibility=hidden", "-ffp-contract=off",
             # no packed-fp32 instructions anywhere in device code
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-I", INCLUDE, "-I", CSRC]
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    tag = "%d" % os.getpid()

    def compile_one(src):
        obj = os.path.join(objdir, os.path.splitext(src)[0] + "." + tag + ".o")
        cmd = flags + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        return obj, r

    with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        results = list(ex.map(compile_one, SOURCES))
    objs = []
    for obj, r in results:
        err = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                        if "packed-fp32-ops" not in l)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + err)
        objs.append(obj)
    tmp = LIB + ".tmp" + tag
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-Wl,--no-undefined",
           "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    for o in objs:
        os.remove(o)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, LIB)
    build_call(tag, verbose)
    return LIB


def build_call(tag, verbose=False):
    """The CPython extension (plain C: it holds no device code)."""
    tmp = CALL + ".tmp" + tag
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-std=gnu11", "-Wall", "-shared", "-fPIC",
           "-fvisibility=hidden", "-D__HIP_PLATFORM_AMD__=1",
           "-I", sysconfig.get_paths()["include"], "-I", INCLUDE,
           "-I", os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"),
           os.path.join(CSRC, "ifq_call.c"), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("ifq_call.c failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, CALL)
    untagged = os.path.join(HERE, "_ifqcall.so")     # of a build for any interpreter
    if os.path.exists(untagged) and untagged != CALL:
        os.remove(untagged)


if __name__ == "__main__":
    print(build(verbose="-q" not in sys.argv))
