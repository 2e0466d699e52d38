"""Builds libk2d.so (the C-ABI library of include/k2d.h) for gfx950 with hipcc, in-tree."""
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
SOURCES = [os.path.join(CSRC, f) for f in ("step_large.hip", "step_medium.hip", "step_small.hip", "k2d.hip")]
HEADERS = [os.path.join(CSRC, f) for f in ("common.h", "step_kernel.h")] + [os.path.join(ROOT, "include", "k2d.h")]
LIB = os.path.join(HERE, "libk2d.so")

# -ffp-contract=off: a*b+c is rounded twice, like a plain evaluation of the paper's formulas.
# -packed-fp32-ops is switched off on purpose (scalar fp32 VALU code only).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-fPIC", "-I" + os.path.join(ROOT, "include")]


LIB_TIMERS = os.path.join(HERE, "libk2d_timers.so")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd))
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed (exit %d):\n%s\n%s" % (r.returncode, r.stdout[-4000:], r.stderr[-8000:]))
    if verbose:
        print(r.stderr)


def build(verbose=False, phase_timers=False):
    """Compiles the library; phase_timers=True builds the instrumented twin (libk2d_timers.so, compiled with
    -DK2D_PHASE_TIMERS: the step kernel records the clocks of its phases) that phase_timers.py uses."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    out = LIB_TIMERS if phase_timers else LIB
    flags = FLAGS + (["-DK2D_PHASE_TIMERS"] if phase_timers else [])
    with tempfile.TemporaryDirectory(dir=HERE, prefix="_build_") as tmp:
        objs = [os.path.join(tmp, os.path.basename(f)[:-4] + ".o") for f in SOURCES]
        with ThreadPoolExecutor(len(SOURCES)) as pool:   # a capacity class of the step kernel per translation unit
            list(pool.map(lambda fo: _run([hipcc] + flags + ["-c", fo[0], "-o", fo[1]], verbose), zip(SOURCES, objs)))
        linked = os.path.join(tmp, "lib.so")
        _run([hipcc, "--offload-arch=gfx950", "-shared", "-o", linked] + objs, verbose)
        os.replace(linked, out)
    return out


def stale():
    """True if the library is missing or older than a source or header."""
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.exists(f) and os.path.getmtime(f) > t for f in SOURCES + HEADERS)


def ensure_built():
    """Path of the built library; rebuilds it when it is missing or older than its sources (where no
    compiler is installed, a library that is there is used as it is)."""
    if stale():
        hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
        if os.path.exists(LIB) and not os.path.exists(hipcc):
            return LIB
        build()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
