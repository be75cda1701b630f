"""Build libeora.so (HIP, gfx950 only) in-tree with hipcc.  Usage: python paper_2410_21271_amd/build.py (run by path: the package itself cannot be imported before the library exists)"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.environ.get("EORA_OBJ_DIR") or os.path.join(HERE, "_build")
LIB = os.environ.get("EORA_LIB_OUT") or os.path.join(HERE, "libeora.so")      # override: debug variants
SOURCES = ["api.hip", "small.hip", "sparse.hip", "wideq.hip", "stream.hip", "prefill.hip", "prefill128.hip", "calibrate.hip", "debug.hip", "pack.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC] + os.environ.get("EORA_EXTRA_FLAGS", "").split()


def _hipcc():
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def _fresh(obj, src):
    """EORA_INCREMENTAL=1 (development): keep an object that is newer than its source and every header."""
    if not os.environ.get("EORA_INCREMENTAL") or os.environ.get("EORA_EXTRA_FLAGS") or not os.path.exists(obj):
        return False
    deps = [os.path.join(CSRC, src)] + [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hpp", ".inc"))]
    deps += [os.path.join(ROOT, "include", f) for f in os.listdir(os.path.join(ROOT, "include"))]
    return all(os.path.getmtime(d) < os.path.getmtime(obj) for d in deps)


# Kernels of these files stream weights at four wavefronts per SIMD with every tile request in flight: an
# instantiation that spills even a few bytes stores freshly requested data to scratch, waits for it first, and runs
# 1.5 to 2 times slower with all tests still passing.  The build therefore reads the compiler's resource remarks
# and refuses an instantiation with a non-zero scratch size.  The GEMM for many tokens counts its requests (x goes to LDS behind the
# compiler's back): a spill's own stores and loads are requests too.
NO_SPILL = {"small.hip": "small_kernel", "stream.hip": "resident_kernel", "prefill.hip": "prefill_kernel"}


def _check_resources(src, remarks):
    name, bad = None, []
    for line in remarks.splitlines():
        m = re.search(r"remark: Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and name and NO_SPILL[src] in name and int(m.group(1)) > 0:
            bad.append("%s: %s bytes of scratch per lane" % (name, m.group(1)))
    if bad:
        raise RuntimeError("%s: register spills in a kernel that must not have any:\n  %s" % (src, "\n  ".join(bad)))


def _compile(src):
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    if _fresh(obj, src):
        return obj
    extra = ["-Rpass-analysis=kernel-resource-usage"] if src in NO_SPILL else []
    cmd = [_hipcc(), *FLAGS, *extra, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, p.stderr[-6000:]))
    if src in NO_SPILL:
        try:
            _check_resources(src, p.stderr)
        except RuntimeError:
            os.remove(obj)
            raise
    return obj


def build(verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    p = subprocess.run(cmd, capture_output=True, text=True)
    if p.returncode:
        raise RuntimeError("link failed:\n" + p.stderr[-6000:])
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
