"""The library's host code on the CPU, over a stand-in for the HIP runtime (_hip_host.c): what an
asynchronous copy reads is still there when the copy runs."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, importlib.util, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
count = lambda name: ctypes.c_int.in_dll(shim, name)
spec = importlib.util.spec_from_file_location("_lib", sys.argv[2] + "/paper_1008_0502_amd/_lib.py")
L = importlib.util.module_from_spec(spec)
spec.loader.exec_module(L)
lib = L.load()
def params(**kw):
    p = L.sp_params()
    lib.sp_default_params(ctypes.byref(p))
    for k, v in kw.items():
        if isinstance(v, tuple):
            setattr(p, "n_" + k, len(v))
            getattr(p, k)[:len(v)] = v
        else:
            setattr(p, k, v)
    return p
def create(H, W, **kw):
    h = ctypes.c_void_p()
    L.check(lib.sp_create(ctypes.byref(params(**kw)), H, W, None, ctypes.byref(h)), "sp_create")
    return h
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("shim") / "libhiphost.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", os.path.join(HERE, "_hip_host.c"), "-o", out], check=True)
    return out


def run(shim, body):
    """The body in a process of its own, after the prelude; it asserts by itself."""
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, shim, ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("tape", [0, 3, 400])
def test_sources_of_copies_outlive_them(shim, tape):
    run(shim, f"""
h = create(96, 128, record_tape={tape})
w = (ctypes.c_float * 8)(*range(8))
L.check(lib.sp_set_weights(h, w, 1e-3, 1e-1), "sp_set_weights")
L.check(lib.sp_set_tune(h, 16, 0, 1), "sp_set_tune")
assert count("shim_pending").value == 0 and count("shim_stale").value == 0, count("shim_stale").value
""")
