"""Kernel launches that fail, on the CPU: a stand-in for the HIP runtime (hip_shim.cpp) counts the launches of a call and
lets one of them fail.  A step whose ordering (keys, then places) did not start must report it and launch nothing that
uses the ordering: the step kernel takes the ordering's entries as record indices, and the counting sort the keys as
indices of its bins."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

CALLS = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before the library: its HIP calls resolve to the stand-in
from paper_2410_23208_amd import binding
import scenegen
lib = binding.lib()
fake = ctypes.c_void_p(0x1000100)                             # never dereferenced: no kernel runs
prm = binding.make_params(scenegen.default_params())
for caps in ((5, 2, 1, 1), (6, 3, 2, 2), (12, 4, 6, 2)):
    c, h = binding.make_caps(caps), ctypes.c_void_p()
    assert lib.k2d_alloc_batch(ctypes.byref(c), ctypes.byref(prm), 40, fake, 1 << 30, ctypes.byref(h)) == 0
    for lanes in (16, 8):
        assert lib.k2d_set_lanes_per_env(h, lanes) == 0
        for call in (lambda n: lib.k2d_step(h, fake, 40, n, None), lambda n: lib.k2d_step_noalloc(h, fake, 40, n, None),
                     lambda n: lib.k2d_step_reset(h, fake, 40, n, fake, 3, fake, None)):
            # an ordered launch (8 steps or more) is keys, places, step; shorter ones are the step alone
            for n, fail_at, rc, launched in ((8, 0, 0, 3), (8, 1, -4, 1), (8, 2, -4, 2), (8, 3, -4, 3), (7, 0, 0, 1), (7, 1, -4, 1)):
                shim.shim_arm(fail_at)
                got = (call(n), shim.shim_launches())
                assert got == (rc, launched), (caps, lanes, n, fail_at, got)
    lib.k2d_free_batch(h)
print("ok")
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("shim") / "libhip_shim.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_shim.cpp")], check=True)
    return so


def test_step_launches_nothing_behind_an_ordering_that_failed(shim):
    r = subprocess.run([sys.executable, "-c", CALLS, shim], cwd=os.path.dirname(HERE), capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stderr[-2000:]
