"""Builds libmipgemm.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import glob
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmipgemm.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def _compile(args):
    hipcc, src, obj = args
    cmd = [hipcc] + [f for f in HIPCC_FLAGS if f != "-shared"] + ["-c", "-x", "hip", src, "-o", obj]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 feature and says so: harmless
    out = "\n".join(l for l in proc.stdout.splitlines() if "packed-fp32-ops" not in l)
    return src, proc.returncode, out


def build_library(verbose: bool = False, jobs: int = 0) -> str:
    """Compile every kernel and the C-ABI layer (one object per source, in parallel) and link."""
    from concurrent.futures import ThreadPoolExecutor
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    work = [(hipcc, src, os.path.join(objdir, os.path.basename(src) + ".o")) for src in sources()]
    jobs = jobs or min(len(work), max(1, min(16, os.cpu_count() or 1)))
    with ThreadPoolExecutor(max_workers=jobs) as pool:
        results = list(pool.map(_compile, work))
    failed = [(src, out) for src, rc, out in results if rc != 0]
    if failed:
        raise RuntimeError("hipcc failed:\n" + "\n".join("%s:\n%s" % f for f in failed))
    if verbose:
        for src, _, out in results:
            print("compiled", os.path.relpath(src, HERE), flush=True)
            if out.strip():
                print(out, flush=True)
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC"] + [w[2] for w in work] + ["-o", tmp]
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("link failed:\n" + proc.stdout)
    os.replace(tmp, LIB)
    build_binding(verbose)
    return LIB


def build_binding(verbose: bool = False) -> bool:
    """The binding's argument conversion (native/call.c), for this interpreter; without Python's headers or a
    C compiler the binding converts its arguments through ctypes."""
    for old in glob.glob(os.path.join(HERE, "_call*.so")):
        os.remove(old)
    include = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(include, "Python.h")):
        print("no Python.h in %s: the binding converts its arguments through ctypes" % include, flush=True)
        return False
    out = os.path.join(HERE, "_call" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
    tmp = out + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CC", "gcc"), "-O2", "-std=c11", "-Wall", "-shared", "-fPIC", "-I" + include,
           os.path.join(HERE, "native", "call.c"), "-o", tmp]
    try:
        proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        failed = proc.stdout if proc.returncode != 0 else None
    except OSError as e:
        failed = str(e)
    if failed is not None:
        if os.path.exists(tmp):
            os.remove(tmp)
        print("native/call.c did not compile, the binding converts its arguments through ctypes:\n" + failed, flush=True)
        return False
    os.replace(tmp, out)
    if verbose:
        print("compiled native/call.c", flush=True)
    return True


if __name__ == "__main__":
    print(build_library(verbose=True))
