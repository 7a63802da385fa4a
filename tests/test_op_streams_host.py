"""Streams and events of the kernel-level calls, without a GPU: a recorder stands in for the HIP runtime and writes down what the
library enqueues where (tests/hip_recorder.cpp)."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2112_09335_amd", "libcadmm.so")

PRELUDE = """
import ctypes, sys
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
rec.recorder_log.restype = ctypes.c_char_p
lib.cadmm_last_error.restype = ctypes.c_char_p
vp, i64, i32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32
lib.cadmm_create.argtypes = [vp, ctypes.c_int, vp]
lib.cadmm_op_stream.argtypes = [vp, vp]
lib.cadmm_op_transform.argtypes = [vp, vp, i64, i32, vp, i32, vp]
lib.cadmm_op_wgrad_noalloc.argtypes = [vp, vp, vp, i64, i32, i32, vp]
lib.cadmm_last_error.argtypes = [vp]
lib.cadmm_destroy.argtypes = [vp]
OWN, A, B = 0x100, 0x200, 0x300
h = vp()
assert lib.cadmm_create(ctypes.byref(h), 0, OWN) == 0

def call(stream, kind="transform"):
    # what one call on `stream` enqueues: its return value and the recorder's lines
    rec.recorder_clear()
    assert lib.cadmm_op_stream(h, stream) == 0
    buf = 0x20000
    rc = lib.cadmm_op_transform(h, buf, 1000, 64, buf, 48, buf) if kind == "transform" else lib.cadmm_op_wgrad_noalloc(h, buf, buf, 1000, 64, 48, buf)
    return rc, [(w, int(a), int(b)) for w, a, b in (l.split() for l in rec.recorder_log().decode().splitlines())]
"""


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    if not os.path.exists(LIB):
        import __graft_entry__
        __graft_entry__.build()
    so = str(tmp_path_factory.mktemp("recorder") / "hip_recorder.so")
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", os.path.join(HERE, "hip_recorder.cpp"), "-o", so], check=True)

    def run(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE + body, so, LIB], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout + r.stderr
    return run


def test_a_call_on_the_null_stream_of_another_device_is_refused_and_runs_nothing(recorder):
    """The null stream is that of the current device: with another one current the call cannot run where the context's memory
    is.  It is an error, and nothing is launched.  (The call without allocation makes the context's device current itself.)"""
    recorder("""
assert call(None)[0] == 0
assert rec.hipSetDevice(1) == 0
for _ in range(2):
    rc, log = call(None)
    assert rc != 0 and b"device" in lib.cadmm_last_error(h), rc
    assert log == [], log
rc, log = call(None, "wgrad")
assert rc == 0 and all(b == 0 for w, a, b in log if w == "launch"), log
rc, log = call(A)                                    # a stream of the caller's: wherever it belongs
assert rc == 0 and ("launch", A, 1) in log, (rc, log)
assert not any(w == "record-elsewhere" for w, a, b in log), log
assert rec.hipSetDevice(0) == 0
assert call(None)[0] == 0
""")


def test_a_call_on_another_stream_waits_for_the_call_before_it_and_not_for_the_null_stream(recorder):
    """Calls on the null stream alone enqueue their kernels and nothing else.  Once a call has gone to another stream, every call has
    its event right behind its kernels: the next one on another stream waits for that event, and records nothing on the null
    stream, where the program's own work may have been enqueued in between."""
    recorder("""
for _ in range(3):
    rc, log = call(None)
    assert rc == 0 and [w for w, _, _ in log] == ["launch"], log
rc, log = call(A)                                    # the first change: the event is recorded now, whatever the thread captures
assert [w for w, _, _ in log] == ["record-relaxed", "wait", "launch", "record"], log
assert log[1] == ("wait", A, log[0][1]) and log[3] == ("record", log[0][1], A)
ev = log[0][1]
for other in (B, OWN, A, A):
    for _ in range(2):
        rc, log = call(None)
        assert log[-2:] == [("launch", 0, 0), ("record", ev, 0)], log
    rc, log = call(other)
    assert log[:2] == [("wait", other, ev), ("launch", other, 0)], log
    assert not any(w.startswith("record") and b == 0 for w, _, b in log), log
""")
