"""Every node of a box belongs to exactly one thread of one column of the
z-marching kernels, whatever the tile's shape against the box's (CPU only:
the host code and the kernels' ownership rule, compiled for the host)."""
import os
import subprocess

import pytest

from paper_2309_07801_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def test_each_node_has_one_owner(tmp_path):
    if not os.path.exists(B.HIPCC):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "column_tiles")
    # (the launch tables live in other units and are never reached)
    subprocess.check_call([B.HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O1",
                           "-std=c++17", "-I", os.path.join(B.ROOT, "include"),
                           "-Wl,--unresolved-symbols=ignore-all", "-o", exe,
                           os.path.join(HERE, "host", "column_tiles.hip")],
                          stderr=subprocess.DEVNULL)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "layouts ok" in r.stdout, r.stdout[-2000:]
