"""Which kernel gives the three-kernel schedule its interface fields (CPU only,
on the stand-in runtime): the fused kernel's export from 2 Mi nodes on, but not
where much of it would run with the logic of y walls; and which kernel the
autotuner times for layouts that the fused kernel does not step."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "host"))
import standin as S  # noqa: E402


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return S.build(tmp_path_factory.mktemp("standin"))


@pytest.mark.parametrize("shapes,export", [
    ([(64, 64, 64, 0)], False), ([(128, 128, 128, 0)], True), ([(32, 32, 32, 0)] * 64, True),
    ([(64, 64, 512, 3)], False), ([(64, 64, 64, 3)] * 8, False), ([(32, 32, 32, 3)] * 64, False),
    ([(1024, 48, 48, 2)], True), ([(256, 128, 128, 3)], True), ([(192, 192, 192, 3)], True)])
def test_interface_fields_of_a_step(lib, shapes, export):
    assert "ok" in S.run(lib, """
import standin as S
h = S.Handle(%r)
h.call("set_schedule", 1, stream=False)
h.call("step", 1)
n = S.standin().standin_launches
assert (n(b"k_interface<") == 0) == %r and (n(b"k_fused<") > 0) == %r
h.close()
assert not S.faults()
print("ok")
""" % (shapes, export, export))


@pytest.mark.parametrize("shape,walls,stored", [((128, 128, 128), 0, False), ((64, 64, 64), 0, True),
                                                ((96, 96, 384), 2, False)])
def test_autotuner_times_what_general_layouts_run(lib, shape, walls, stored):
    """Rates other than one: no population-storing fused kernel in large boxes."""
    assert "ok" in S.run(lib, """
import standin as S
h = S.Handle([%r + (%d,)], omega_hi=(1.2,) * 9)
h.call("autotune", 2, None)
L = S.standin()
# (k_fused<geometry, waves, walls, storage, export, compact, plain>)
stores = sum(L.standin_launches(("StoreF32, false, false, " + p).encode()) for p in ("true", "false"))
exports = L.standin_launches(b"StoreF32, true, false, false")
assert (stores > 0) == %r and (exports > 0) == (not %r), (stores, exports)
h.close()
assert not S.faults()
print("ok")
""" % (shape, walls, stored, stored))
