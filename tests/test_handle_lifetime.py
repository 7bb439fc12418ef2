"""Graphs, events and streams of a handle are destroyed only when no work on
them is pending, and events before the streams they were recorded on: handles
with and without walls that step, are re-tuned, change their schedule and close
while the steps may still be running (CPU only, on the stand-in runtime, which
notes every violation)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "host"))
import standin as S  # noqa: E402


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return S.build(tmp_path_factory.mktemp("standin"))


SCRIPT = """
import standin as S
for walls in (0, 3):
    for schedule in (0, 1, 2):
        for change in ("destroy", "set_schedule", "set_variant", "set_wall_mode",
                       "set_compact_variant", "autotune", "set_resident"):
            h = S.Handle([(40, 24, 30, walls)])
            h.call("set_schedule", schedule, stream=False)
            if change == "set_resident":
                h.call("set_resident", 1)
            h.call("step", 7)
            if change == "set_schedule":
                for k in range(40):
                    h.call("set_schedule", (schedule + 1 + k) % 3, stream=False)
                    h.call("step", 5)
            elif change == "autotune":
                h.call("autotune", 2, None)
            elif change != "destroy":
                h.call(change, 2 if change != "set_resident" else 0)
            h.call("step", 6)
            h.close()
            bad = S.faults()
            assert not bad, (walls, schedule, change, bad)
print("ok")
"""


def test_nothing_is_destroyed_while_work_on_it_is_pending(lib):
    assert "ok" in S.run(lib, SCRIPT)


def test_walled_handles_one_after_another_under_other_streams(lib):
    """Handles on streams of their own, several alive at once, closed in the
    order they were opened; the caller's streams outlive them."""
    assert "ok" in S.run(lib, """
import standin as S, ctypes as C
L = S.standin()
streams = []
for k in range(3):
    p = C.c_void_p()
    L.hipStreamCreateWithFlags(C.byref(p), 0)
    streams.append(p)
alive = []
for k in range(12):
    h = S.Handle([(33, 17 + k, 20, k % 4), (12, 9, 8, 0)], stream=streams[k % 3])
    if k % 2:
        h.call("autotune", 1, None)
        h.call("set_schedule", 2, stream=False)
    h.call("step", 8)
    alive.append(h)
    if len(alive) > 3:
        alive.pop(0).close()
for h in alive:
    h.close()
bad = S.faults()
assert not bad, bad
print("ok")
""")
