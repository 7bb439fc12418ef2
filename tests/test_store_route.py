"""Which population stores a step's fused kernel makes (CPU only, on the
stand-in runtime): streaming ones where a row of stored words is whole cache
lines, or beyond 128 nodes whole 64-byte sectors, plain ones elsewhere; a batch
goes by where most of its nodes lie."""
import os
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.abspath(__file__)), "host"))
import standin as S  # noqa: E402

FP32, FP16, EXACT, PAIRS = 0, 1, 3, 4


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return S.build(tmp_path_factory.mktemp("standin"))


@pytest.mark.parametrize("nx,storage,plain", [
    ([64], FP32, False), ([256], FP16, False), ([200], EXACT, False), ([200], PAIRS, False),
    ([240], FP32, False), ([136], EXACT, False), ([112], FP32, True), ([72], PAIRS, True),
    ([200], FP32, True), ([197], EXACT, True), ([200], FP16, True), ([33], FP32, True),
    ([200, 64, 64], FP32, True), ([200, 256], FP32, False)])
def test_population_stores(lib, nx, storage, plain):
    assert "ok" in S.run(lib, """
import standin as S
h = S.Handle([(n, 20, 18, 0) for n in %r], storage=%d)
h.call("step", 1)
# (k_fused<geometry, waves, walls, storage, export, compact, plain>)
n = [sum(S.standin().standin_launches(("Store%%s, false, false, %%s>" %% (s, p)).encode())
         for s in ("F32", "F16", "F32X", "F32P")) for p in ("false", "true")]
assert n == ([0, 1] if %r else [1, 0]), n
h.close()
print("ok")
""" % (nx, storage, plain))
