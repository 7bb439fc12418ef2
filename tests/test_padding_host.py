"""The padding of the population buffers is zeroed once after the compact
schedule's arrays lay in one, before the next steps of another schedule, and
under a caller's capture without being taken for done (CPU only, on the
stand-in runtime; what the kernel does is tests/test_gpu_padding.py)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "host"))
import standin as S  # noqa: E402


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return S.build(tmp_path_factory.mktemp("standin"))


def test_padding_is_zeroed_once(lib):
    assert "ok" in S.run(lib, """
import ctypes as C
import standin as S
L = S.standin()
n = lambda: L.standin_launches(b"k_zero_pad<")
h = S.Handle([(40, 24, 30, 0), (33, 17, 20, 3)])
h.call("step", 5)
assert n() == 0
h.call("autotune", 1, None)
assert n() == 0
h.call("step", 0)
assert n() == 0
for k in range(3):
    h.call("step", 5)
assert n() == 1
h.call("set_schedule", 2, stream=False)
h.call("step", 5)
h.call("step", 5)
h.call("set_schedule", 1, stream=False)
h.call("step", 1)
h.call("step", 1)
assert n() == 2
# captured by the caller: recorded, and still to be done
h.call("set_graph", 0, stream=False)
h.call("set_schedule", 2, stream=False)
h.call("step", 2)
h.call("set_schedule", 0, stream=False)
s = C.c_void_p()
L.hipStreamCreateWithFlags(C.byref(s), 0)
L.hipStreamBeginCapture(s, 0)
h.ok(h.L.cglbm_step(h.h, 2, s))
g = C.c_void_p()
L.hipStreamEndCapture(s, C.byref(g))
assert n() == 3
h.call("step", 2)
h.call("step", 2)
assert n() == 4
# a captured call of the compact schedule may be replayed at any time
h.call("set_schedule", 2, stream=False)
L.hipStreamBeginCapture(s, 0)
h.ok(h.L.cglbm_step(h.h, 2, s))
L.hipStreamEndCapture(s, C.byref(g))
h.call("set_schedule", 0, stream=False)
h.call("step", 2)
h.call("step", 2)
assert n() == 6
h.close()
assert not S.faults()
print("ok")
""")
