"""The library's host code on the CPU, over a stand-in for the HIP runtime (_hip_host.c): what an
asynchronous copy reads is still there when the copy runs; launch tables that could not be made anew
leave the old ones in use; clips are queued without waiting for the ones before,
and take forced launch shapes; the allocation-free call takes the frames that it took."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, importlib.util, sys
standin = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
count = lambda name: ctypes.c_int.in_dll(standin, name)
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
def standin(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("standin") / "libhiphost.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", os.path.join(HERE, "_hip_host.c"), "-o", out], check=True)
    return out


def run(standin, body):
    """The body in a process of its own, after the prelude; it asserts by itself."""
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, standin, ROOT], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("tape", [0, 3, 400])
def test_sources_of_copies_outlive_them(standin, tape):
    run(standin, f"""
h = create(96, 128, record_tape={tape})
w = (ctypes.c_float * 8)(*range(8))
L.check(lib.sp_set_weights(h, w, 1e-3, 1e-1), "sp_set_weights")
L.check(lib.sp_set_tune(h, 16, 0, 1), "sp_set_tune")
assert count("standin_pending").value == 0 and count("standin_stale").value == 0, count("standin_stale").value
""")


STEP = """
JOB = 8 * 4
def launches(call):
    "grid, threads and (where its first argument is a job table) the jobs of every launch of a call"
    n0 = count("standin_launches").value
    call()
    standin.standin_launch.restype = ctypes.POINTER(ctypes.c_uint * 4)
    out = []
    for i in range(n0, count("standin_launches").value):
        r = standin.standin_launch(i).contents
        jobs = r[2] | r[3] << 32
        out.append((r[0], r[1], ctypes.string_at(jobs, r[0] * JOB)))
    return out
def mem(n):
    bufs.append(ctypes.create_string_buffer(n))
    return ctypes.addressof(bufs[-1])
bufs = []
"""


@pytest.mark.parametrize("fault", ["malloc", "copy"])
def test_refused_tables_keep_the_context(standin, fault):
    run(standin, STEP + f"""
h = create(721, 1000)
rgb, S, P = mem(721 * 1000 * 3), mem(4 * 721 * 1000), mem(4 * 721 * 1000)
def step():
    L.check(lib.sp_step(h, rgb, None, None, S, None, P, None, None, None), "sp_step")
L.check(lib.sp_set_tune(h, 64, 0, 4), "sp_set_tune")
before = launches(step)
count("standin_fail_{fault}").value = 1
assert lib.sp_set_tune(h, 16, 1, 1) != 0
count("standin_fail_{fault}").value = 0
assert launches(step) == before and before
L.check(lib.sp_set_tune(h, 16, 1, 1), "sp_set_tune")
assert launches(step) != before
""")


def test_refused_tables_keep_the_batch(standin):
    run(standin, STEP + """
b = ctypes.c_void_p()
dims = (ctypes.c_int32 * 2)(96, 120), (ctypes.c_int32 * 2)(128, 97)
L.check(lib.sp_batch_create(ctypes.byref(params(record_tape=3)), 2, *dims, 0, None, ctypes.byref(b)), "sp_batch_create")
L.check(lib.sp_batch_profile_enable(b, 1), "sp_batch_profile_enable")   # steps by launches, not a graph
tab = (ctypes.c_void_p * 2)(mem(96 * 128 * 3), mem(120 * 97 * 3))
def step():
    L.check(lib.sp_batch_step(b, ctypes.cast(tab, ctypes.c_void_p), None), "sp_batch_step")
L.check(lib.sp_batch_set_tune(b, 64, 0, 8), "sp_batch_set_tune")
before = launches(step)
count("standin_fail_copy").value = 1
assert lib.sp_batch_set_tune(b, 16, 1, 1) != 0
count("standin_fail_copy").value = 0
assert launches(step) == before and before
L.check(lib.sp_batch_set_tune(b, 16, 1, 1), "sp_batch_set_tune")
assert launches(step) != before
""")


def test_clips_are_queued_without_a_wait(standin):
    run(standin, STEP + """
H, W, T = 48, 64, 5
h = create(H, W, record_tape=T)
n = H * W
frames = [mem(3 * n) for _ in range(T)]
clip = mem(3 * n * T)
table = (ctypes.c_void_p * T)(*frames)
S, P, U, PW, B, G, gw, gf = (mem(4 * k * n * T) for k in (1, 1, 2, 4, 1, 1, 1, 3))
def clips(k):
    for _ in range(k):
        L.check(lib.sp_run_clip(h, table, T, None, S, None, P, U, PW, B), "sp_run_clip")
w0 = count("standin_waits").value
clips(4)
assert count("standin_waits").value == w0 and count("standin_pending").value == 0
L.check(lib.saliency_backward(h, G, T, gw, gw + 64, gw + 128), "saliency_backward")
w0 = count("standin_waits").value
for _ in range(3):
    L.check(lib.saliency_backward_frames(h, clip, T, gf), "saliency_backward_frames")
assert count("standin_waits").value == w0 and count("standin_pending").value == 0
""")


def test_forced_shapes_reach_the_clip(standin):
    run(standin, STEP + """
H, W, T = 120, 160, 6
h = create(H, W, record_tape=T)
n = H * W
table = (ctypes.c_void_p * T)(*[mem(3 * n) for _ in range(T)])
S, P = mem(4 * n * T), mem(4 * n * T)
def clip():
    L.check(lib.sp_run_clip(h, table, T, None, S, None, P, None, None, None), "sp_run_clip")
def shaped(xcd, channels):
    L.check(lib.sp_set_tune(h, 16, xcd, channels), "sp_set_tune")
    return [j for _, _, j in launches(clip) if j]
a, b, c = shaped(1, 1), shaped(1, 4), shaped(0, 4)
assert len(a) == len(b) == len(c)
assert sum(map(len, b)) < sum(map(len, a))                      # fewer across-scale workgroups
cut = lambda j: sorted(j[i:i + JOB] for i in range(0, len(j), JOB))
assert b != c and [cut(x) for x in b] == [cut(x) for x in c]     # the same jobs in another order
""")


@pytest.mark.parametrize("levels,H,W", [(dict(depth=9, centers=(2, 3, 4), deltas=(3, 4)), 1080, 8968),
                                        (dict(depth=9, centers=(2, 3, 4), deltas=(3, 4)), 1501, 6448),
                                        (dict(depth=8, centers=(3, 4), deltas=(3,)), 2000, 5514),
                                        (dict(depth=9, centers=(4,), deltas=(3, 4, 5)), 2160, 5216)])
def test_largest_frames_without_allocation(standin, levels, H, W):
    """The largest width at this height whose scratch fits with two channels a workgroup; the next does not."""
    run(standin, STEP + f"""
p, buf = params(**{levels}), mem(64)
call = lambda W: lib.sp_saliency_noalloc(ctypes.byref(p), {H}, W, buf, None, buf, None, None)
assert call({W}) == L.SP_OK, lib.sp_last_error()
assert call({W} + 16) == L.SP_ESHAPE
""")
