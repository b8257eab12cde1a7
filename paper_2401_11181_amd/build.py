"""Build libtetri.so (HIP, gfx950 only) in-tree with hipcc, and the CPython module _native.so that calls it."""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtetri.so")
NATIVE = os.path.join(HERE, "_native.so")
SOURCES = ["tetri_host.cpp", "tetri_plan.cpp", "tetri_append.hip", "tetri_kv_transfer.hip", "tetri_decode.hip", "tetri_attn.hip", "tetri_planned.hip", "tetri_short.hip"]
HEADERS = [os.path.join(CSRC, "tetri_internal.h"), os.path.join(CSRC, "tetri_plan.h"), os.path.join(CSRC, "attn_common.h"), os.path.join(CSRC, "attn_tile.h"), os.path.join(ROOT, "include", "tetri.h")]

# packed-fp32 instructions are switched off for all device code; a kernel's leading scalar arguments (up to 14 words in front of
# its first structure) are in registers when a wavefront starts, instead of a first memory read away
HIP_FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
             "-mllvm", "-amdgpu-kernarg-preload-count=16",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-Wno-unused-command-line-argument", "-Wno-ignored-attributes"]


def hipcc():
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.isabs(cand) and os.path.exists(cand) or not os.path.isabs(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def build(force=True, verbose=False, extra_flags=()):
    """Compile every source and link libtetri.so.  Returns its path."""
    objs, jobs = [], []
    for src in SOURCES:                              # compiled side by side
        path = os.path.join(CSRC, src)
        obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
        deps = [path] + HEADERS
        if force or not os.path.exists(obj) or any(os.path.getmtime(d) > os.path.getmtime(obj) for d in deps):
            cmd = [hipcc(), "-x", "hip", "-c", path, "-o", obj, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                   "-DTETRI_BUILDING=1"] + HIP_FLAGS + list(extra_flags)
            if verbose:
                print(" ".join(cmd), flush=True)
            jobs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)))
        objs.append(obj)
    failed = []
    for src, job in jobs:
        noise = "is not a recognized feature for this target"
        err = "\n".join(l for l in job.communicate()[1].splitlines() if noise not in l)
        if job.returncode != 0:
            failed.append("hipcc failed for %s:\n%s" % (src, err))
        elif err.strip() and verbose:
            print(err, file=sys.stderr)
    if failed:
        raise RuntimeError("\n".join(failed))
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    build_native(verbose)
    return LIB


def build_native(verbose=False):
    """Compile the CPython module of fast calls (host code only).  Returns its path."""
    cmd = [os.environ.get("CXX", "g++"), "-std=c++17", "-O2", "-shared", "-fPIC", "-fvisibility=hidden", "-Wno-cast-function-type",
           "-I", sysconfig.get_paths()["include"], "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "tetri_py.cpp"), "-o", NATIVE, "-ldl"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("compiling tetri_py.cpp failed:\n" + res.stderr)
    return NATIVE


if __name__ == "__main__":
    print(build(force="--incremental" not in sys.argv, verbose=True))
